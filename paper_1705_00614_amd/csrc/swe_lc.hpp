// swe_lc.hpp -- gfx950 kernels of the learned coarse-grid flux correction.
//
// A small convolutional network (four 3x3 valid convolutions, 6 -> 32 -> 32
// -> 32 -> 6 channels, tanh after the first three) reads the state of a
// coarse grid and predicts corrections of the stage III face fluxes (Sec. 2.3
// of arXiv 1705.00614; the learned part is an extension of the method, the
// paper has none).  The network runs on crops: for an active S x S tile the
// (S+9)^2 window round the tile and the cell row and column before it
// (mirrored at walls) gives the (S+1)^2 corrections of those cells, so that
// the tile's west and south boundary faces (east and north faces of the
// neighbours' cells) are always fresh.
//
// Layouts: activations bf16, [crop][y][x][C] with C = 16 (the 6 features,
// zero padded) or 32; weights bf16 as [tap][out][in] (forward) and
// [tap][in][out] (backward data), both padded to multiples of 16; FP32 master
// weights, gradients and Adam moments in the packed order (W[out][in][3][3],
// then b[out]) per layer.  Every contraction is a 16x16x16 bf16 MFMA with
// FP32 accumulation: a wave owns 16 consecutive pixels (M) of one crop and
// all output channels (N tiles of 16), the reduction (K) runs over the 9 taps
// times the input channels in chunks of 16.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swe {
namespace lc {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NL = 4;                         // layers
constexpr int HALO = NL;                      // crop margin
constexpr int CIN[NL] = {16, 32, 32, 32};     // padded input channels
constexpr int COUT[NL] = {32, 32, 32, 16};    // padded output channels
constexpr int CIN_REAL[NL] = {6, 32, 32, 32};
constexpr int COUT_REAL[NL] = {32, 32, 32, 6};

// packed FP32 parameter offsets of layer l: W then b (offsets by loops, which
// unroll where a kernel's layer loop does; as recursions they were calls)
__host__ __device__ constexpr int w_count(int l) { return COUT_REAL[l] * CIN_REAL[l] * 9; }
__host__ __device__ constexpr int p_off(int l) {
    int o = 0;
    for (int q = 0; q < l; ++q) o += w_count(q) + COUT_REAL[q];
    return o;
}
constexpr int NPARAM = p_off(NL);
// bf16 weight copies: [tap][COUT][CIN] per layer
__host__ __device__ constexpr int wb_count(int l) { return 9 * COUT[l] * CIN[l]; }
__host__ __device__ constexpr int wb_off(int l) {
    int o = 0;
    for (int q = 0; q < l; ++q) o += wb_count(q);
    return o;
}
constexpr int NWB = wb_off(NL);
// block partials of the weight gradients: layer l has at most PART_BLOCKS of
// part_elems(l) floats ([tap][COUT][CIN], then [COUT]), of at least 16 pixels
// each; part_blocks(px) is the most that batches of up to px pixels have
constexpr int PART_BLOCKS = 512;
inline int part_blocks(long long px) { return (int)((px + 15) / 16 < PART_BLOCKS ? (px + 15) / 16 : PART_BLOCKS); }
__host__ __device__ constexpr int part_elems_of(int ci, int co) { return 9 * co * ci + co; }
__host__ __device__ constexpr int part_elems(int l) { return part_elems_of(CIN[l], COUT[l]); }

__device__ __forceinline__ unsigned short to_bf16(float f) {
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
// Two values rounded to nearest even as bf16, packed (one instruction).
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{lo, hi}), b16x2));
}
__device__ __forceinline__ float from_bf16(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

__device__ __forceinline__ bf16x4 load4(const unsigned short* p) {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    bf16x4 r;
    r[0] = (short)(v.x & 0xFFFFu);
    r[1] = (short)(v.x >> 16);
    r[2] = (short)(v.y & 0xFFFFu);
    r[3] = (short)(v.y >> 16);
    return r;
}

// Number of crops: from the device (active tiles of a grid) or the host.
__device__ __forceinline__ int crop_count(const int* dev, int host) { return dev ? *dev : host; }

// ------------------------------------------------------------------ forward
// y = act(conv3x3_valid(x) + b); x [n][Sin][Sin][CI] bf16, y [n][Sout][Sout][CO]
// (bf16 with tanh, or FP32 linear for the last layer).
//
// A wave keeps the layer's weights for every tap and output tile in registers
// for all its items, and loads the pixels of its next 16-pixel item while the
// MFMAs of the current one run.  With 32 input channels a tap is one 16x16x32
// bf16 MFMA (lane group kq holds channels 8kq..8kq+7 of both operands, one
// 16-byte load each); with 16 input channels a tap is one 16x16x16 MFMA.  The
// weights are the first operand, so that a lane ends up with four consecutive
// channels of one pixel.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 as8(const uint4& q) { return __builtin_bit_cast(bf16x8, q); }

// tanh of the hidden activations (stored as bf16): an odd Taylor polynomial
// below 1/16, else 1 - 2 / (e^(2|x|) + 1) from the hardware base-2 exponential
// and reciprocal; relative error about 1e-6, far below the bf16 spacing.
__device__ __forceinline__ float tanh_act(float x) {
    const float ax = __builtin_fabsf(x), x2 = x * x;
    const float small = x * (1.f + x2 * (-0.333333343f + x2 * 0.133333340f));
    const float e = __builtin_amdgcn_exp2f(2.88539008f * ax);
    const float big = __builtin_copysignf(1.f - 2.f * __builtin_amdgcn_rcpf(e + 1.f), x);
    return ax < 0.0625f ? small : big;
}

template <int CI> struct AFrag;
template <> struct AFrag<16> { typedef uint2 Q; Q v[9]; };
template <> struct AFrag<32> { typedef uint4 Q; Q v[9]; };

__device__ __forceinline__ bf16x4 as4(const uint2& q) {
    bf16x4 r;
    r[0] = (short)(q.x & 0xFFFFu); r[1] = (short)(q.x >> 16); r[2] = (short)(q.y & 0xFFFFu); r[3] = (short)(q.y >> 16);
    return r;
}

template <int CI>
__device__ __forceinline__ void load_a(AFrag<CI>& f, const unsigned short* __restrict__ x, int item, int blocks,
                                       int Sin, int Sout, int P, int m, int kq) {
    const int c = item / blocks, p = min((item % blocks) * 16 + m, P - 1);
    const int oy = p / Sout, ox = p % Sout;
    const unsigned short* xc = x + (size_t)c * Sin * Sin * CI;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const unsigned short* xp = xc + ((oy + tap / 3) * Sin + ox + tap % 3) * CI;
        if constexpr (CI == 32) f.v[tap] = *reinterpret_cast<const uint4*>(xp + 8 * kq);
        else f.v[tap] = *reinterpret_cast<const uint2*>(xp + 4 * kq);
    }
}

template <int CI, int CO, bool LAST>
__global__ __launch_bounds__(256) void k_conv_fwd(const unsigned short* __restrict__ x, void* __restrict__ y,
                                                   const unsigned short* __restrict__ wf, const float* __restrict__ bias,
                                                   int cob, int Sin, const int* cnt_dev, int cnt_host) {
    static_assert(CI == 16 || CI == 32, "input channels");
    constexpr int NT = CO / 16;
    const int Sout = Sin - 2, P = Sout * Sout, blocks = (P + 15) / 16;
    const int n = crop_count(cnt_dev, cnt_host);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int m = lane & 15, kq = lane >> 4;
    const int total = n * blocks, stride = gridDim.x * 4;
    int item = blockIdx.x * 4 + wv;
    if (item >= total) return;
    // weights: lane (m, kq) holds w[tap][t*16 + m][k] for its k of each chunk,
    // as the pixels' operand holds x[pixel m][k]
    typename AFrag<CI>::Q B[9][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
            B[tap][t] = *reinterpret_cast<const typename AFrag<CI>::Q*>(wf + (tap * CO + t * 16 + m) * CI +
                                                                         (CI / 4) * kq);
    float bb[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) bb[t][i] = t * 16 + 4 * kq + i < cob ? bias[t * 16 + 4 * kq + i] : 0.f;
    AFrag<CI> cur, nxt;
    load_a<CI>(cur, x, item, blocks, Sin, Sout, P, m, kq);
    for (; item < total; item += stride) {
        const int item2 = item + stride;
        if (item2 < total) load_a<CI>(nxt, x, item2, blocks, Sin, Sout, P, m, kq);
        f32x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (CI == 32)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as8(B[tap][t]), as8(cur.v[tap]), acc[t], 0, 0, 0);
                else
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as4(B[tap][t]), as4(cur.v[tap]), acc[t], 0, 0, 0);
            }
        // lane: pixel p0 + m, channels t * 16 + 4 * kq + i, stored together
        const int c = item / blocks, pp = (item % blocks) * 16 + m;
        if (pp < P) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int ch = t * 16 + 4 * kq;
                const size_t o = ((size_t)c * P + pp) * CO + ch;
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = acc[t][i] + bb[t][i];
                if constexpr (LAST)
                    *reinterpret_cast<float4*>(static_cast<float*>(y) + o) =
                        float4{ch < cob ? v[0] : 0.f, ch + 1 < cob ? v[1] : 0.f, ch + 2 < cob ? v[2] : 0.f,
                               ch + 3 < cob ? v[3] : 0.f};
                else
                    *reinterpret_cast<uint2*>(static_cast<unsigned short*>(y) + o) =
                        uint2{pack_bf16(tanh_act(v[0]), tanh_act(v[1])), pack_bf16(tanh_act(v[2]), tanh_act(v[3]))};
            }
        }
        cur = nxt;
    }
}

// ------------------------------------------------------------------ fused inference
// All four layers of one T x T block of a crop's output in one workgroup, the
// intermediate activations in LDS: the block's (T+8)^2 input window comes in
// from HBM once and only the FP32 output goes out, so an inference costs one
// launch instead of four and no activation round trips through HBM.  The
// weights of the two middle layers are staged in LDS once per workgroup, the
// smaller ones of the outer layers go from L2 to registers; that leaves LDS
// for two workgroups per CU, whose MFMAs, activations and LDS reads overlap
// (each alone takes 2 to 3 us of a block).  Each layer is the same per-pixel
// MFMA sequence as k_conv_fwd (taps in order, one MFMA per tap and output
// tile, the same bias, tanh and bf16 rounding), with the operands exchanged so
// that a lane holds four channels of a pixel and stores them together; the
// output equals the layer-by-layer forward.  A crop of side So is covered by
// ceil(So / T) blocks per side, the last one shifted back to end at So (its
// overlap is recomputed and written with the same values).
constexpr int w_elems(int l) { return 9 * COUT[l] * CIN[l]; }
template <int T>
struct alignas(16) NetLds {
    static constexpr int P16 = 24, P32 = 40;      // pixel strides (bf16): channels + 8 against bank conflicts
    // a hidden layer's output plane is padded to whole 16-pixel blocks, so
    // that the rows of a ragged last block are stored without a test (and
    // never read)
    static constexpr int blk16(int side) { return ((side * side + 15) / 16) * 16; }
    static constexpr int A = (T + 8) * (T + 8) * P16 > blk16(T + 4) * P32 ? (T + 8) * (T + 8) * P16
                                                                           : blk16(T + 4) * P32;
    static constexpr int B = blk16(T + 6) * P32;
    unsigned short w[w_elems(1) + w_elems(2)];    // bf16 weights of layers 1 and 2, [tap][CO][CI]
    float bias[NL][32];
    unsigned short a[A];                          // input window, then layer-1 output
    unsigned short b[B];                          // layer-0 output, then layer-2 output
};

// The thread's lane, opaque to the compiler: the addresses made from it are
// not kept in registers over a workgroup's units (they would spill).
__device__ __forceinline__ int opaque_lane() {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    return tid & 63;
}

// A layer's weights as MFMA operands: lane m + 16 kq holds channels
// (CI / 4) kq .. of output channel t * 16 + m, for every tap.
template <int CI, int CO>
struct WFrag {
    typename AFrag<CI>::Q v[9][CO / 16];
    __device__ __forceinline__ void load(const unsigned short* w) {
        const int lane = opaque_lane(), m = lane & 15, kq = lane >> 4;
#pragma unroll
        for (int t = 0; t < CO / 16; ++t)
#pragma unroll
            for (int tap = 0; tap < 9; ++tap)
                v[tap][t] = *reinterpret_cast<const typename AFrag<CI>::Q*>(w + (tap * CO + t * 16 + m) * CI +
                                                                           (CI / 4) * kq);
    }
};

// One layer over the LDS plane `in` (side Win, pixel stride PI) into `out`
// (LDS bf16 with tanh, stride PO) or, for the last layer, through the writer
// `wr(oy, ox, ch, v)` (block-local output pixel, channel, FP32 value).
struct NoWriter {
    __device__ __forceinline__ void operator()(int, int, int, float) const {}
};
template <int CI, int CO, bool LAST, int Win, int NTH, class Wr>
__device__ __forceinline__ void net_layer(const unsigned short* in, int PI, unsigned short* out, int PO,
                                          const WFrag<CI, CO>& W, const float* bias, int cob, const Wr& wr) {
    constexpr int NT = CO / 16, Wout = Win - 2, P = Wout * Wout, blocks = (P + 15) / 16, nw = NTH / 64;
    const int lane = opaque_lane(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, kq = lane >> 4;
#pragma unroll 1
    for (int blk = wv; blk < blocks; blk += nw) {
        const int pix = blk * 16 + m, p = min(pix, P - 1);
        const int oy = p / Wout, ox = p % Wout;
        const unsigned short* ip = in + (oy * Win + ox) * PI + (CI / 4) * kq;
        f32x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            const typename AFrag<CI>::Q av =
                *reinterpret_cast<const typename AFrag<CI>::Q*>(ip + ((tap / 3) * Win + tap % 3) * PI);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (CI == 32)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as8(W.v[tap][t]), as8(av), acc[t], 0, 0, 0);
                else
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as4(W.v[tap][t]), as4(av), acc[t], 0, 0, 0);
            }
        }
        // lane: pixel blk * 16 + m, channels t * 16 + 4 * kq + i
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int ch = t * 16 + 4 * kq;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = acc[t][i] + bias[ch + i];
            if constexpr (LAST) {
                if (pix < P) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) wr(oy, ox, ch + i, ch + i < cob ? v[i] : 0.f);
                }
            } else {   // pix < blocks * 16: inside the padded plane
                *reinterpret_cast<uint2*>(out + pix * PO + ch) =
                    uint2{pack_bf16(tanh_act(v[0]), tanh_act(v[1])), pack_bf16(tanh_act(v[2]), tanh_act(v[3]))};
            }
        }
    }
}

// A workgroup's share (blockIdx.x, then every gridDim.x-th) of `units` blocks
// through the four layers.  The source `src` (a read-only descriptor; what it
// fetches is held in three 16-byte registers of the caller, plain locals so
// that they stay in VGPRs) provides the input windows and the output writers:
//   src.find(u, s)             the thread that knows unit u's id writes it to *s,
//   src.load(id, q0, q1, q2)   fetch a unit's input window,
//   src.store(lds, q0, q1, q2) put it into the LDS plane (pixel stride 24),
//   src.writer(id)             the last layer's writer.
// The next unit's window is fetched while the current one computes.
template <int T, int NTH, class Src>
__device__ __forceinline__ void net_run(const Src& src, NetLds<T>& L, const unsigned short* __restrict__ wf,
                                        const float* __restrict__ params, int units) {
    using N = NetLds<T>;
    if ((int)blockIdx.x >= units) return;
    const int tid = threadIdx.x;
    constexpr int W0 = T + 2 * HALO;
    __shared__ int s_unit;
    src.find((int)blockIdx.x, &s_unit);
    // every global load of the weight staging is issued before the first
    // store (one memory round trip, not one per piece)
    {
        constexpr int NV = (w_elems(1) + w_elems(2)) / 8, J = (NV + NTH - 1) / NTH;
        static_assert(wb_off(2) == wb_off(1) + w_elems(1), "layers 1 and 2 follow each other");
        uint4 v[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k = min(tid + j * NTH, NV - 1);   // clamped: the tail re-reads the last piece
            v[j] = reinterpret_cast<const uint4*>(wf + wb_off(1))[k];
        }
#pragma unroll
        for (int j = 0; j < J; ++j)
            if (tid + j * NTH < NV) reinterpret_cast<uint4*>(L.w)[tid + j * NTH] = v[j];
    }
    for (int k = tid; k < NL * 32; k += NTH) {
        const int l = k / 32, ch = k % 32;
        constexpr int b0 = p_off(0) + w_count(0), b1 = p_off(1) + w_count(1), b2 = p_off(2) + w_count(2),
                      b3 = p_off(3) + w_count(3);   // bias offsets, folded at compile time
        const int off = l == 0 ? b0 : l == 1 ? b1 : l == 2 ? b2 : b3;
        L.bias[l][ch] = ch < (l == NL - 1 ? COUT_REAL[NL - 1] : 32) ? params[off + ch] : 0.f;
    }
    __syncthreads();
    int id = __builtin_amdgcn_readfirstlane(s_unit);
    uint4 q0, q1, q2;
    src.load(id, q0, q1, q2);
    for (int u = blockIdx.x;; ) {
        WFrag<16, 32> w0;
        w0.load(wf + wb_off(0));
        src.store(L.a, q0, q1, q2);
        __syncthreads();
        const int un = u + (int)gridDim.x, cur = id;
        if (un < units) src.find(un, &s_unit);
        const NoWriter nw;
        net_layer<16, 32, false, W0, NTH>(L.a, N::P16, L.b, N::P32, w0, L.bias[0], 32, nw);
        __syncthreads();
        if (un < units) {
            id = __builtin_amdgcn_readfirstlane(s_unit);
            src.load(id, q0, q1, q2);
        }
        {
            WFrag<32, 32> w;
            w.load(L.w);
            net_layer<32, 32, false, W0 - 2, NTH>(L.b, N::P32, L.a, N::P32, w, L.bias[1], 32, nw);
            __syncthreads();
            w.load(L.w + w_elems(1));
            net_layer<32, 32, false, W0 - 4, NTH>(L.a, N::P32, L.b, N::P32, w, L.bias[2], 32, nw);
        }
        WFrag<32, 16> w3;
        w3.load(wf + wb_off(3));
        __syncthreads();
        net_layer<32, 16, true, W0 - 6, NTH>(L.b, N::P32, nullptr, 0, w3, L.bias[3], COUT_REAL[3], src.writer(cur));
        // the next unit's input goes to L.a, last read by layer 2 (before the
        // barrier above); layer 3 reads L.b, next written after the barrier
        // that follows the next input
        if (un >= units) break;
        u = un;
    }
}

// Writer of the last layer into the FP32 crop output y [n][So][So][16].
struct CropWriter {
    float* y;
    int So, c, oy0, ox0;
    __device__ __forceinline__ void operator()(int oy, int ox, int ch, float v) const {
        y[(((size_t)c * So + oy0 + oy) * So + ox0 + ox) * 16 + ch] = v;
    }
};

// Source of crops already in HBM: x [n][So+8][So+8][16] bf16; each thread
// moves two 16-byte pieces (tid and tid + NTH) of the window.
template <int T, int NTH>
struct CropSource {
    static constexpr int W0 = T + 2 * HALO, XV = W0 * W0 * 2;
    static_assert(XV > NTH && XV <= 2 * NTH, "two 16-byte pieces of the input window per thread");
    const unsigned short* x;
    float* y;
    int So, ns, tid;
    __device__ __forceinline__ int origin(int u, int& oy0, int& ox0) const {
        const int sub = u % (ns * ns);
        oy0 = min((sub / ns) * T, So - T);
        ox0 = min((sub % ns) * T, So - T);
        return u / (ns * ns);
    }
    __device__ __forceinline__ void find(int u, int* s) const { if (tid == 0) *s = u; }
    __device__ __forceinline__ void load(int u, uint4& q0, uint4& q1, uint4&) const {
        int oy0, ox0;
        const int Sin = So + 2 * HALO, c = origin(u, oy0, ox0);
        const unsigned short* xc = x + (size_t)c * Sin * Sin * 16;
        const int k0 = tid, k1 = tid + NTH;
        q0 = *reinterpret_cast<const uint4*>(xc + ((size_t)(oy0 + (k0 >> 1) / W0) * Sin + ox0 + (k0 >> 1) % W0) *
                                                        16 + 8 * (k0 & 1));
        if (k1 < XV)
            q1 = *reinterpret_cast<const uint4*>(xc + ((size_t)(oy0 + (k1 >> 1) / W0) * Sin + ox0 + (k1 >> 1) % W0) *
                                                          16 + 8 * (k1 & 1));
    }
    __device__ __forceinline__ void store(unsigned short* a, const uint4& q0, const uint4& q1, const uint4&) const {
        *reinterpret_cast<uint4*>(a + (tid >> 1) * NetLds<T>::P16 + 8 * (tid & 1)) = q0;
        if (tid + NTH < XV) *reinterpret_cast<uint4*>(a + ((tid + NTH) >> 1) * NetLds<T>::P16 + 8 * (tid & 1)) = q1;
    }
    __device__ __forceinline__ CropWriter writer(int u) const {
        int oy0, ox0;
        const int c = origin(u, oy0, ox0);
        return CropWriter{y, So, c, oy0, ox0};
    }
};

// x: crops [n][So+8][So+8][16] bf16; y: [n][So][So][16] FP32 (channels >= 6
// zero); wf: bf16 weights of all layers; params: packed FP32 parameters (the
// biases are read from there).  Requires So >= T; n from the device or host.
constexpr int NET_WAVES = 4;   // waves per SIMD of the fused kernels: two workgroups of 512 threads per CU
template <int T, int NTH>
__global__ __launch_bounds__(NTH, NET_WAVES) void k_net_fwd(const unsigned short* __restrict__ x, float* __restrict__ y,
                                                 const unsigned short* __restrict__ wf,
                                                 const float* __restrict__ params, int So, const int* cnt_dev,
                                                 int cnt_host) {
    __shared__ NetLds<T> L;
    const int ns = (So + T - 1) / T;
    const CropSource<T, NTH> src{x, y, So, ns, (int)threadIdx.x};
    net_run<T, NTH>(src, L, wf, params, crop_count(cnt_dev, cnt_host) * ns * ns);
}

// ------------------------------------------------------------------ backward data
// g_in = bf16(dL/da_in * (1 - a_in^2)) from g = dL/dz of this layer:
// dL/da_in[q] = sum_{tap, co} g[q - tap][co] w[co][ci][tap] (zero outside the
// output plane).  a_in and g_in: [n][Sin][Sin][CI]; g: [n][Sout][Sout][CO].
//
// As in the forward, a wave keeps the layer's weights (of every tap and
// 16-channel chunk) in registers for all its 16-pixel items and loads the
// next item's gradients and activations while the current one's MFMAs run.
template <int CI, int CO>
struct BwdItem {
    uint2 g[9][CO / 16];
    uint2 a[CI / 16];
    int in;      // taps inside the output plane, one bit each
};
template <int CI, int CO>
__device__ __forceinline__ void load_bwd(BwdItem<CI, CO>& f, const unsigned short* __restrict__ g,
                                         const unsigned short* __restrict__ a_in, int item, int blocks, int Sin, int P,
                                         int m, int kq) {
    const int Sout = Sin - 2, c = item / blocks, p = min((item % blocks) * 16 + m, P - 1);
    const int qy = p / Sin, qx = p % Sin;
    const unsigned short* gc = g + (size_t)c * Sout * Sout * CO + 4 * kq;
    f.in = 0;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
        const int oy = qy - tap / 3, ox = qx - tap % 3;
        const bool in = oy >= 0 && oy < Sout && ox >= 0 && ox < Sout;
        f.in |= in << tap;
        const unsigned short* gp = gc + ((in ? oy : 0) * Sout + (in ? ox : 0)) * CO;
#pragma unroll
        for (int h = 0; h < CO / 16; ++h) f.g[tap][h] = *reinterpret_cast<const uint2*>(gp + 16 * h);
    }
#pragma unroll
    for (int t = 0; t < CI / 16; ++t)
        f.a[t] = *reinterpret_cast<const uint2*>(a_in + ((size_t)c * P + p) * CI + t * 16 + 4 * kq);
}

template <int CI, int CO>
__global__ __launch_bounds__(256) void k_conv_bwd_data(const unsigned short* __restrict__ g,
                                                        const unsigned short* __restrict__ a_in,
                                                        unsigned short* __restrict__ g_in,
                                                        const unsigned short* __restrict__ wb, int Sin, int n) {
    constexpr int NT = CI / 16, NH = CO / 16;
    const int P = Sin * Sin, blocks = (P + 15) / 16, total = n * blocks, stride = gridDim.x * 4;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int m = lane & 15, kq = lane >> 4;
    int item = blockIdx.x * 4 + wv;
    if (item >= total) return;
    uint2 B[9][NH][NT];
#pragma unroll
    for (int tap = 0; tap < 9; ++tap)
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                B[tap][h][t] = *reinterpret_cast<const uint2*>(wb + (tap * CI + t * 16 + m) * CO + 16 * h + 4 * kq);
    BwdItem<CI, CO> cur, nxt;
    load_bwd<CI, CO>(cur, g, a_in, item, blocks, Sin, P, m, kq);
    for (; item < total; item += stride) {
        if (item + stride < total) load_bwd<CI, CO>(nxt, g, a_in, item + stride, blocks, Sin, P, m, kq);
        f32x4 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int tap = 0; tap < 9; ++tap)
#pragma unroll
            for (int h = 0; h < NH; ++h) {
                bf16x4 a = as4(cur.g[tap][h]);
                if (!((cur.in >> tap) & 1)) a = bf16x4{0, 0, 0, 0};
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as4(B[tap][h][t]), a, acc[t], 0, 0, 0);
            }
        // lane: pixel p0 + m, channels t * 16 + 4 * kq + i
        const int c = item / blocks, pp = (item % blocks) * 16 + m;
        if (pp < P) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const bf16x4 a4 = as4(cur.a[t]);
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = from_bf16((unsigned short)a4[i]);
                    v[i] = acc[t][i] * (1.f - a * a);
                }
                *reinterpret_cast<uint2*>(g_in + ((size_t)c * P + pp) * CI + t * 16 + 4 * kq) =
                    uint2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            }
        }
        cur = nxt;
    }
}

// ------------------------------------------------------------------ backward weights
// Partial weight and bias gradients of one pixel chunk per block:
// dW[tap][co][ci] = sum_p g[p][co] a_in[p + tap][ci], db[co] = sum_p g[p][co].
// part[block] holds [tap][CO][CI] then [CO] in FP32; the chunk's pixels enter
// in order, 16 per MFMA.
//
// The reduction runs over pixels, but both operands lie channels-last, so an
// MFMA lane (4 pixels of one channel) is a column of 4 rows.  The chunk's g
// rows and the a_in rows its taps reach are staged in LDS as they lie (both
// are contiguous in memory), WG_SUB pixels at a time, and read back through
// the transposing LDS load: a group of 16 lanes reads 4 pixel rows of 16
// channels at any 4 row addresses, so a tap is a constant offset and chunks
// cross rows and crops freely.  Reading each operand element by 2-byte global
// loads instead took 96 us for a 32 -> 32 layer of 64 crops of 39^2 and 291 us
// for the four layers (one launch each); this takes 24.7 us for all of them,
// bound by its 57 MB of partials.
constexpr int WG_SUB = 96;     // pixels staged at a time
constexpr int WG_NTH = 320;    // four MFMA waves and one for the bias sums
// Positions of the input plane between the first pixel of `sub` consecutive
// outputs (side so) and the last one's last tap: one per pixel, two more per
// row end and 2 (so + 2) more per crop end passed.
__host__ __device__ constexpr int wg_span(int so, int sub) {
    const int d = sub - 1, si = so + 2;
    return d + 2 * (d / so + 1) + 2 * si * (d / (so * so) + 1) + 2 * si + 3;
}
constexpr int WG_SPAN = 400;
constexpr bool wg_span_fits() {
    for (int so = 2; so <= 64 + 1 + 2 * (NL - 1); ++so)   // output sides of tiles of 1 to 64 cells
        if (wg_span(so, WG_SUB) > WG_SPAN) return false;
    return true;
}
static_assert(wg_span_fits(), "a sub-chunk's input rows must fit their LDS buffer");

struct alignas(16) WgLds {
    unsigned short g[WG_SUB * 32];
    unsigned short a[WG_SPAN * 32];
    int off[WG_SUB];           // element offset of each pixel's first tap in a[]
};

__device__ __forceinline__ bf16x4 lds_column(const unsigned short* p) {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_bf16x4*)p);
}

template <int CI, int CO>
__device__ __forceinline__ void wgrad_chunk(WgLds& L, const unsigned short* __restrict__ g,
                                            const unsigned short* __restrict__ a_in, float* __restrict__ part, int Sin,
                                            int n, int chunk, int blk) {
    constexpr int TCO = CO / 16, TCI = CI / 16, NC = TCO * TCI, PARTS = 4 / NC, TP = (9 + PARTS - 1) / PARTS;
    const int Sout = Sin - 2, P = Sout * Sout, total = n * P;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int q0 = blk * chunk, q1 = min(total, q0 + chunk);
    // wave -> output channels (to, ti) and its share of the taps
    const int to = (wv % NC) / TCI, ti = wv % TCI, tap0 = (wv / NC) % PARTS;
    auto pos = [&](int q) {
        const int c = q / P, p = q % P;
        return (c * Sin + p / Sout) * Sin + p % Sout;
    };
    f32x4 acc[TP];
#pragma unroll
    for (int j = 0; j < TP; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;
    for (int s0 = q0; s0 < q1; s0 += WG_SUB) {
        const int cnt = min(WG_SUB, q1 - s0), rows = (cnt + 15) / 16 * 16;
        const int base = pos(s0), len = pos(s0 + cnt - 1) + 2 * Sin + 3 - base;
        __syncthreads();   // the previous sub-chunk is read
        {
            const uint4* src = reinterpret_cast<const uint4*>(g + (size_t)s0 * CO);
            uint4* dst = reinterpret_cast<uint4*>(L.g);
            for (int k = tid; k < rows * CO / 8; k += WG_NTH) dst[k] = k < cnt * CO / 8 ? src[k] : uint4{0u, 0u, 0u, 0u};
        }
        {
            const uint4* src = reinterpret_cast<const uint4*>(a_in + (size_t)base * CI);
            uint4* dst = reinterpret_cast<uint4*>(L.a);
            for (int k = tid; k < len * CI / 8; k += WG_NTH) dst[k] = src[k];
        }
        // pixels past the chunk have g = 0 and read the first pixel's taps
        if (tid < rows) L.off[tid] = tid < cnt ? (pos(s0 + tid) - base) * CI : 0;
        __syncthreads();
        if (wv < 4) {
            const int r = (lane >> 4) * 4 + ((lane & 15) >> 2), c4 = (lane & 3) * 4;
            for (int k0 = 0; k0 < rows; k0 += 16) {
                const bf16x4 av = lds_column(L.g + (k0 + r) * CO + to * 16 + c4);
                const unsigned short* ap = L.a + L.off[k0 + r] + ti * 16 + c4;
#pragma unroll
                for (int j = 0; j < TP; ++j) {
                    const int tap = tap0 + PARTS * j;
                    if (TP * PARTS > 9 && tap >= 9) break;
                    const bf16x4 bv = lds_column(ap + ((tap / 3) * Sin + tap % 3) * CI);
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv, acc[j], 0, 0, 0);
                }
            }
        } else if (lane < CO) {   // bias: each lane sums its channel over the chunk
#pragma unroll 8
            for (int q = 0; q < cnt; ++q) bsum += from_bf16(L.g[q * CO + lane]);
        }
    }
    float* out = part + (size_t)blk * part_elems_of(CI, CO);
    const int m = lane & 15, kq = lane >> 4;
    if (wv < 4) {
        // lane holds rows (co) to*16 + 4*kq + i, column (ci) ti*16 + m
#pragma unroll
        for (int j = 0; j < TP; ++j) {
            const int tap = tap0 + PARTS * j;
            if (TP * PARTS > 9 && tap >= 9) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) out[(tap * CO + to * 16 + 4 * kq + i) * CI + ti * 16 + m] = acc[j][i];
        }
    } else if (lane < CO) {
        out[9 * CO * CI + lane] = bsum;
    }
}

// All layers in one launch (after the backward-data passes): nblk[l] chunks
// of layer l.
struct WgradArgs {
    const unsigned short* g[NL];
    const unsigned short* a[NL];
    float* part[NL];
    int nblk[NL], chunk[NL];
    int Sin0, n;               // input side of layer 0, crops
};
__global__ __launch_bounds__(WG_NTH) void k_conv_bwd_w(WgradArgs w) {
    __shared__ WgLds L;
    int b = blockIdx.x;
    if (b < w.nblk[1])
        return wgrad_chunk<32, 32>(L, w.g[1], w.a[1], w.part[1], w.Sin0 - 2, w.n, w.chunk[1], b);
    b -= w.nblk[1];
    if (b < w.nblk[2])
        return wgrad_chunk<32, 32>(L, w.g[2], w.a[2], w.part[2], w.Sin0 - 4, w.n, w.chunk[2], b);
    b -= w.nblk[2];
    if (b < w.nblk[0])
        return wgrad_chunk<16, 32>(L, w.g[0], w.a[0], w.part[0], w.Sin0, w.n, w.chunk[0], b);
    b -= w.nblk[0];
    wgrad_chunk<32, 16>(L, w.g[3], w.a[3], w.part[3], w.Sin0 - 6, w.n, w.chunk[3], b);
}

// ------------------------------------------------------------------ parameters
// bf16 copies of the packed FP32 weights in both layouts (zero padding).
__global__ void k_pack_weights(const float* __restrict__ params, unsigned short* __restrict__ wf,
                               unsigned short* __restrict__ wb) {
    for (int l = 0; l < NL; ++l) {
        const int ci_p = CIN[l], co_p = COUT[l], cir = CIN_REAL[l], cor = COUT_REAL[l];
        const float* W = params + p_off(l);
        for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < 9 * co_p * ci_p; k += gridDim.x * blockDim.x) {
            const int tap = k / (co_p * ci_p), co = (k / ci_p) % co_p, ci = k % ci_p;
            const float v = (co < cor && ci < cir) ? W[(co * cir + ci) * 9 + tap] : 0.f;
            const unsigned short h = to_bf16(v);
            wf[wb_off(l) + (tap * co_p + co) * ci_p + ci] = h;
            wb[wb_off(l) + (tap * ci_p + ci) * co_p + co] = h;
        }
    }
}

// ------------------------------------------------------------------ gradient sums and Adam
constexpr int OPT_E = 64;        // gradient elements per workgroup (one per lane)
constexpr int OPT_ROWS = 128;    // block partials staged at a time
constexpr int OPT_NTH = 512;
__host__ __device__ constexpr int opt_blocks(int l) { return (part_elems(l) + OPT_E - 1) / OPT_E; }
constexpr int OPT_GRID = opt_blocks(0) + opt_blocks(1) + opt_blocks(2) + opt_blocks(3) + 1;

struct OptArgs {
    const float* part[NL];      // block partials of each layer
    int nblk[NL];               // and their number
    float *params, *grads, *m, *v;
    unsigned short *wf, *wb;    // bf16 weight copies [tap][out][in] and [tap][in][out]
    const double* loss_part;    // loss partials of the batch, their count, and the loss
    int loss_blocks;
    double* loss;
    int adam;                   // 0: gradient (and loss) only
    float lr, b1, b2, eps, c1, c2;
};

// The end of an optimisation step in one launch: every gradient element is
// the sum of its block partials in block order (the order is part of the
// result: FP32 sums), then its Adam update (bias-corrected) and its bf16
// weight copies, all of which are elementwise in the parameter; the last
// workgroup sums the loss partials in order.  A workgroup owns 64 elements:
// its eight waves fetch the partials of 128 blocks at a time (16 coalesced
// 256-byte rows per wave in flight) into LDS while wave 0 adds the previous
// 128, so the serial chain is LDS reads and adds, not memory round trips.
// 64 crops of a 32-cell tile (498 to 512 partials a layer): one thread per
// element with its loads in the chain took 151-309 us per layer (four
// launches, 928 us) plus Adam, packing and a host sum of the loss; this takes
// 12 us, reading the 57 MB of partials at 4.8 TB/s.
__global__ __launch_bounds__(OPT_NTH) void k_opt(OptArgs a) {
    constexpr int NW = OPT_NTH / 64, J = OPT_ROWS / NW;
    __shared__ float buf[2][OPT_ROWS][OPT_E];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int l = 0, blk = blockIdx.x;
#pragma unroll
    for (int q = 0; q < NL; ++q)
        if (l == q && blk >= opt_blocks(q)) { blk -= opt_blocks(q); l = q + 1; }
    if (l == NL) {   // the loss
        __shared__ double lp[OPT_NTH];
        double s = 0.0;
        for (int k0 = 0; k0 < a.loss_blocks; k0 += OPT_NTH) {
            const int n = min(OPT_NTH, a.loss_blocks - k0);
            __syncthreads();
            if (tid < n) lp[tid] = a.loss_part[k0 + tid];
            __syncthreads();
            if (tid == 0)
                for (int k = 0; k < n; ++k) s += lp[k];
        }
        if (tid == 0) *a.loss = s;
        return;
    }
    int co_p = 0, ci_p = 0, co_r = 0, ci_r = 0, po = 0, wo = 0, nb = 0;
    const float* part = nullptr;
#pragma unroll
    for (int q = 0; q < NL; ++q)
        if (l == q) {
            co_p = COUT[q]; ci_p = CIN[q]; co_r = COUT_REAL[q]; ci_r = CIN_REAL[q];
            po = p_off(q); wo = wb_off(q); nb = a.nblk[q]; part = a.part[q];
        }
    const int wcount = 9 * co_p * ci_p, per = wcount + co_p;
    const int e = blk * OPT_E + lane;
    const bool has = e < per;
    const float* col = part + (has ? e : 0);
    float r[J];
    auto fetch = [&](int row0) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int b = row0 + wv + NW * j;
            r[j] = b < nb ? col[(size_t)b * per] : 0.f;
        }
    };
    float s = 0.f;
    fetch(0);
    for (int row0 = 0, p = 0; row0 < nb; row0 += OPT_ROWS, p ^= 1) {
#pragma unroll
        for (int j = 0; j < J; ++j) buf[p][wv + NW * j][lane] = r[j];
        __syncthreads();   // also: wave 0 is done with this buffer's previous rows
        if (row0 + OPT_ROWS < nb) fetch(row0 + OPT_ROWS);
        if (wv == 0) {
            const int n = min(OPT_ROWS, nb - row0);
            int k = 0;
            for (; k + 16 <= n; k += 16) {
                float t[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) t[j] = buf[p][k + j][lane];
#pragma unroll
                for (int j = 0; j < 16; ++j) s += t[j];
            }
            for (; k < n; ++k) s += buf[p][k][lane];
        }
    }
    if (wv != 0 || !has) return;
    int k, tap = 0, co = 0, ci = 0;
    const bool weight = e < wcount;
    if (weight) {
        tap = e / (co_p * ci_p); co = (e / ci_p) % co_p; ci = e % ci_p;
        if (co >= co_r || ci >= ci_r) return;   // padding
        k = po + (co * ci_r + ci) * 9 + tap;
    } else {
        if (e - wcount >= co_r) return;
        k = po + co_r * ci_r * 9 + (e - wcount);
    }
    a.grads[k] = s;
    if (!a.adam) return;
    const float gk = s;
    const float mk = a.b1 * a.m[k] + (1.f - a.b1) * gk;
    const float vk = a.b2 * a.v[k] + (1.f - a.b2) * gk * gk;
    a.m[k] = mk;
    a.v[k] = vk;
    float pk = a.params[k];
    pk -= a.lr * (mk / a.c1) / (sqrtf(vk / a.c2) + a.eps);
    a.params[k] = pk;
    if (weight) {
        const unsigned short h = to_bf16(pk);
        a.wf[wo + (tap * co_p + co) * ci_p + ci] = h;
        a.wb[wo + (tap * ci_p + ci) * co_p + co] = h;
    }
}

// ------------------------------------------------------------------ loss
// g = bf16(mask (out - y) / count) for the 6 real channels (zero padding to
// 16); per-block loss partials 1/2 sum mask (out - y)^2 / count.
// Optimisation steps on 4, 64, 160 and 400 crops of a 32-cell tile: with 256
// workgroups 58, 119, 201 and 417 us, with 512 58, 116, 193 and 400, with 1024
// (as launched) 60, 114, 189 and 390; one element at a time in place of J the
// same within 1 %.
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ out, const float* __restrict__ y, const float* __restrict__ mask,
                       unsigned short* __restrict__ g, int npix, float inv_count, double* __restrict__ part) {
    __shared__ double red[4];
    double s = 0.0;
    // (the stride is a multiple of 16: a thread keeps its channel); the loads
    // of J elements go together, their sum in order
    constexpr int J = 5;
    const int n = npix * 16, nt = gridDim.x * blockDim.x, ch = threadIdx.x % 16;
    for (int k0 = blockIdx.x * blockDim.x + threadIdx.x; k0 < n; k0 += J * nt) {
        float o[J], t[J], w[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k = k0 + j * nt;
            const bool in = ch < 6 && k < n;
            o[j] = in ? out[k] : 0.f;
            t[j] = in ? y[k / 16 * 6 + ch] : 0.f;
            w[j] = in ? mask[k / 16 * 6 + ch] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int k = k0 + j * nt;
            if (k >= n) break;
            float gv = 0.f;
            if (ch < 6) {
                const float d = o[j] - t[j], mk = w[j];
                gv = mk * d * inv_count;
                s += 0.5 * (double)(mk * d * d) * (double)inv_count;
            }
            g[k] = to_bf16(gv);
        }
    }
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

}  // namespace lc
}  // namespace swe

// ------------------------------------------------------------------ coarse grid I/O
// These need the step kernel's argument block and tile list.
#include "swe_step.hpp"

namespace swe {
namespace lc {

// Crop p of the grid's current tile list (all tiles when the grid does not
// skip dry tiles).
template <typename real>
__device__ __forceinline__ int crop_tile(const Args<real>& a, int slot, int p) {
    return a.skip ? entry_tile(list_entry(a.ctrl, a.lists, a.ntiles, slot, p)) : p;
}

// Grid cell (mirrored at walls) of pixel (wx, wy) of a tile's (S+9)^2 input
// window, which starts HALO + 1 cells before the tile.
template <typename real>
__device__ __forceinline__ int crop_cell(const Args<real>& a, int tile, int S, int wx, int wy) {
    int fx = 0, fy = 0;
    const int gx = mirror((tile % a.ntx) * S - 1 - HALO + wx, a.nx, fx);
    const int gy = mirror((tile / a.ntx) * S - 1 - HALO + wy, a.ny, fy);
    return gy * a.nx + gx;
}

// The stored values of one cell and its six network features (depth,
// velocity, bed, sqrt(c_f / g) = Manning n, wet flag), divided by the input
// scales, as bf16.
template <typename real> struct CellIn { real H, qx, qy, b, cf; };
template <typename real>
__device__ __forceinline__ void features(const Args<real>& a, const CellIn<real>& v, const float* iscale,
                                         unsigned short (&o)[6]) {
    const bool w = v.H > a.eps;
    float f[6];
    f[0] = (float)v.H;
    f[1] = w ? (float)(v.qx / v.H) : 0.f;
    f[2] = w ? (float)(v.qy / v.H) : 0.f;
    f[3] = (float)v.b;
    f[4] = sqrtf((float)v.cf / (float)a.g_d);
    f[5] = w ? 1.f : 0.f;
#pragma unroll
    for (int c = 0; c < 6; ++c) o[c] = to_bf16(f[c] / iscale[c]);
}

// Input crops of the active tiles: the six features of every cell of each
// (S+9)^2 window (mirrored at walls), divided by the input scales, as bf16.
template <typename real>
__global__ void k_gather(Args<real> a, int slot, int S, const float* __restrict__ iscale, unsigned short* __restrict__ x,
                         int* __restrict__ tiles_out) {
    const int Sin = S + 1 + 2 * HALO, P = Sin * Sin;
    const int n = a.skip ? a.ctrl->seg_off[slot][NSEG] : a.ntiles;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n * P; k += gridDim.x * blockDim.x) {
        const int p = k / P, q = k % P;
        const int tile = crop_tile(a, slot, p);
        if (tiles_out && q == 0) tiles_out[p] = tile;
        const int gi = crop_cell(a, tile, S, q % Sin, q / Sin);
        const CellIn<real> v{a.Hi[gi], a.Qxi[gi], a.Qyi[gi], a.bed[gi], a.cf[gi]};
        unsigned short f[6];
        features(a, v, iscale, f);
        unsigned short* o = x + (size_t)k * 16;
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = f[c];
    }
}

// Corrections of the active tiles' cells and of the cell row and column
// before each tile, from the network output.  A cell shared by two active
// crops gets the same value from both (same inputs, same summation order).
template <typename real>
__global__ void k_scatter(Args<real> a, int slot, int S, const float* __restrict__ oscale, const float* __restrict__ out,
                          real* __restrict__ corrE, real* __restrict__ corrN) {
    const int So = S + 1, P = So * So, nc = a.nx * a.ny;
    const int n = a.skip ? a.ctrl->seg_off[slot][NSEG] : a.ntiles;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n * P; k += gridDim.x * blockDim.x) {
        const int p = k / P, q = k % P;
        const int tile = crop_tile(a, slot, p);
        const int gx = (tile % a.ntx) * S - 1 + q % So, gy = (tile / a.ntx) * S - 1 + q / So;
        if (gx < 0 || gy < 0 || gx >= a.nx || gy >= a.ny) continue;
        const int gi = gy * a.nx + gx;
        const float* o = out + (size_t)k * 16;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            corrE[c * nc + gi] = (real)(o[c] * oscale[c]);
            corrN[c * nc + gi] = (real)(o[3 + c] * oscale[3 + c]);
        }
    }
}

// Writer of the last layer straight into a grid's correction planes (what
// k_scatter does from the crop output): crop pixel (oy0 + oy, ox0 + ox) is
// grid cell (x0 + ox, y0 + oy), x0 = tile column * S - 1 + ox0.
template <typename real>
struct CorrWriter {
    real* corrE;
    real* corrN;
    const float* oscale;
    int nx, ny, x0, y0;
    __device__ __forceinline__ void operator()(int oy, int ox, int ch, float v) const {
        const int gx = x0 + ox, gy = y0 + oy;
        if (ch >= 6 || gx < 0 || gy < 0 || gx >= nx || gy >= ny) return;
        const size_t nc = (size_t)nx * ny, gi = (size_t)gy * nx + gx;
        if (ch < 3) corrE[ch * nc + gi] = (real)(v * oscale[ch]);
        else corrN[(ch - 3) * nc + gi] = (real)(v * oscale[ch]);
    }
};

// The blocks of a grid's active tiles whose corrections some face can take,
// found before the network runs, so that its workgroups share just these (two
// thirds of the blocks of a flood lie in shallow water; tested by the
// network's workgroups, each block skipped cost one 3 to 4 us of dependent
// round trips).  A block runs if one of its output cells or their face
// neighbours is deeper than the correction depth -- the step corrects a face
// only where its cells are -- or lies in the inlet rectangle (the depth that
// decides is the one after the Lagrangian stage, which is the stored one
// except on source cells).  A block not run keeps older corrections, which
// the step never applies there.  Workgroup w of the grid (at most NET_SEGS)
// takes the tiles at list positions w, w + gridDim.x, ... and writes its
// blocks (tile * ns^2 + block) into its own segment of `units`, their number
// into units[w]: nothing to clear, and no order but the list's.  With J loads
// together in place of one, a learned step takes 37.7 in place of 38.9 us on
// 256^2 cells, 43.0 in place of 44.3 on 1024^2, 56.5 in place of 57.8 on 2048^2.
constexpr int NET_SEGS = 512;
constexpr int NET_MAX_SIDE = 5;   // blocks per side whose squares fit a mask word
__host__ __device__ constexpr int net_seg_cap(int ntiles, int ns) { return (ntiles + NET_SEGS - 1) / NET_SEGS * ns * ns; }
template <int T, typename real>
__global__ __launch_bounds__(256) void k_net_units(Args<real> a, int slot, int S, int ns, int cap,
                                                   int* __restrict__ units) {
    __shared__ unsigned s_mask[2];
    const int tid = threadIdx.x, So = S + 1, W = So + 2, P = W * W;
    const int n = a.skip ? a.ctrl->seg_off[slot][NSEG] : a.ntiles;
    int* const seg = units + NET_SEGS + blockIdx.x * cap;
    int cnt = 0;
    if (tid < 2) s_mask[tid] = 0u;
    __syncthreads();
    for (int p = blockIdx.x, it = 0; p < n; p += gridDim.x, it ^= 1) {
        const int tile = __builtin_amdgcn_readfirstlane(crop_tile(a, slot, p));
        unsigned mask = 0u;
        constexpr int J = 5;
        for (int k0 = tid; k0 < P; k0 += 256 * J) {
            real h[J];
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int k = min(k0 + 256 * j, P - 1);   // (the last pixel again)
                h[j] = a.Hi[crop_cell(a, tile, S, HALO - 1 + k % W, HALO - 1 + k / W)];
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int k = min(k0 + 256 * j, P - 1), x = k % W, y = k / W;
                if (!(h[j] > a.corr_hmin)) continue;
                unsigned mx = 0u;
                for (int q = 0; q < ns; ++q) {
                    const int o = min(q * T, So - T);
                    if (x >= o && x <= o + T + 1) mx |= 1u << q;
                }
                for (int q = 0; q < ns; ++q) {
                    const int o = min(q * T, So - T);
                    if (y >= o && y <= o + T + 1) mask |= mx << (q * ns);
                }
            }
        }
        mask = (unsigned)wave_or((int)mask);
        if ((tid & 63) == 0 && mask) atomicOr(&s_mask[it], mask);
        __syncthreads();
        if (tid < 64) {
            bool run = false;
            if (tid < ns * ns) {
                // the block's first face neighbour
                const int x0 = (tile % a.ntx) * S - 2 + min((tid % ns) * T, So - T);
                const int y0 = (tile / a.ntx) * S - 2 + min((tid / ns) * T, So - T);
                const bool source = a.ni > 0 && a.nj > 0 && x0 < a.i0 + a.ni && a.i0 < x0 + T + 2 &&
                                    y0 < a.j0 + a.nj && a.j0 < y0 + T + 2;
                run = source || (s_mask[it] >> tid & 1u);
            }
            const unsigned long long m = __ballot(run);
            if (run) seg[cnt + __popcll(m & ((1ull << tid) - 1))] = tile * ns * ns + tid;
            cnt += __popcll(m);
            // (this word is added to again after the next barrier only)
            if (tid == 0) s_mask[it] = 0u;
        }
    }
    if (tid == 0) units[blockIdx.x] = cnt;
}

// Source of the input windows straight from a grid's current layer (what
// k_gather does into HBM): thread tid < (T+8)^2 fetches the five stored
// values of one window pixel and turns them into its features at the store.
// Thread w holds the range [lo, hi) of units in segment w of k_net_units.
template <int T, int NTH, typename real>
struct GridSource {
    static constexpr int W0 = T + 2 * HALO;
    static_assert(W0 * W0 <= NTH, "one window pixel per thread");
    static_assert(5 * sizeof(real) <= 48, "five stored values in three 16-byte registers");
    const Args<real>* a;
    int S, So, ns, tid;
    const float* iscale;
    real* corrE;
    real* corrN;
    const float* oscale;
    const int* seg;
    int lo, hi;
    __device__ __forceinline__ void find(int u, int* s) const { if (u >= lo && u < hi) *s = seg[u - lo]; }
    __device__ __forceinline__ int origin(int id, int& oy0, int& ox0) const {
        const int sub = id % (ns * ns);
        oy0 = min((sub / ns) * T, So - T);
        ox0 = min((sub % ns) * T, So - T);
        return id / (ns * ns);
    }
    __device__ __forceinline__ void load(int id, uint4& q0, uint4& q1, uint4& q2) const {
        if (tid >= W0 * W0) return;
        int oy0, ox0;
        const int tile = origin(id, oy0, ox0);
        const int gi = crop_cell(*a, tile, S, ox0 + tid % W0, oy0 + tid / W0);
        real v[6] = {a->Hi[gi], a->Qxi[gi], a->Qyi[gi], a->bed[gi], a->cf[gi], real(0)};
        uint4 q[3];
        static_assert(sizeof v <= sizeof q, "fits");
        __builtin_memcpy(q, v, sizeof v);
        q0 = q[0]; q1 = q[1]; q2 = q[2];
    }
    __device__ __forceinline__ void store(unsigned short* lds, const uint4& q0, const uint4& q1, const uint4& q2) const {
        if (tid >= W0 * W0) return;
        const uint4 q[3] = {q0, q1, q2};
        real v[6];
        __builtin_memcpy(v, q, sizeof v);
        unsigned short f[6];
        features(*a, CellIn<real>{v[0], v[1], v[2], v[3], v[4]}, iscale, f);
        const uint4 lo4 = {f[0] | ((unsigned)f[1] << 16), f[2] | ((unsigned)f[3] << 16), f[4] | ((unsigned)f[5] << 16), 0u};
        *reinterpret_cast<uint4*>(lds + tid * NetLds<T>::P16) = lo4;
        *reinterpret_cast<uint4*>(lds + tid * NetLds<T>::P16 + 8) = uint4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ CorrWriter<real> writer(int id) const {
        int oy0, ox0;
        const int tile = origin(id, oy0, ox0);
        return CorrWriter<real>{corrE, corrN, oscale, a->nx, a->ny, (tile % a->ntx) * S - 1 + ox0,
                                (tile / a->ntx) * S - 1 + oy0};
    }
};

// Before a step of a grid with an attached network, after k_net_units: crops
// of the blocks it lists, the four layers and the corrections in one launch
// (the work of k_gather, the four forward layers and k_scatter, with the same
// arithmetic per value).  Requires S + 1 >= T and nseg <= NTH segments.
// 1024 x 1024 cells with 85 active tiles (303 of 765 blocks to run): one
// workgroup per CU that tested its blocks itself and claimed further ones took
// 37.6 us a step; k_net_units 5.4 and this 19.3 us, nearly all of it one
// block's chain (list, window, four layers), as 303 blocks start at once.
template <int T, int NTH, typename real>
__global__ __launch_bounds__(NTH, NET_WAVES) void k_net_grid(Args<real> a, int S, const float* __restrict__ iscale,
                                                             const float* __restrict__ oscale, real* __restrict__ corrE,
                                                             real* __restrict__ corrN,
                                                             const unsigned short* __restrict__ wf,
                                                             const float* __restrict__ params,
                                                             const int* __restrict__ units, int nseg, int cap) {
    static_assert(NET_SEGS <= NTH, "a segment per thread");
    __shared__ NetLds<T> L;
    __shared__ int s_wave[NTH / 64];
    // units before segment tid, and in all
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int mine = tid < nseg ? units[tid] : 0;
    int hi = mine, before = 0, total = 0;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(hi, o, 64);
        if (lane >= o) hi += v;
    }
    if (lane == 63) s_wave[wv] = hi;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NTH / 64; ++q) {
        const int v = s_wave[q];
        if (q < wv) before += v;
        total += v;
    }
    hi += before;
    const int So = S + 1;
    const GridSource<T, NTH, real> src{&a,   S,     So,    (So + T - 1) / T, tid, iscale, corrE, corrN,
                                       oscale, units + NET_SEGS + tid * cap, hi - mine, hi};
    net_run<T, NTH>(src, L, wf, params, __builtin_amdgcn_readfirstlane(total));
}

// Training labels of n crops (coarse tiles tiles[p], (S+1)^2 cells from the
// row and column before the tile): the correction that
// makes each coarse face carry the fine solution's flux over one coarse step,
// (mean of the r fine line taps through the face - the coarse tap) / tau_c,
// divided by the output scales; mask 1 on interior faces of in-domain cells.
// Fine taps: ftx [3][r*ny][nx+1], fty [3][ny+1][r*nx]; coarse taps (r = 1):
// ctx [3][ny][nx+1], cty [3][ny+1][nx] (planes mass, normal, tangential).
template <typename real>
__global__ void k_labels(const int* __restrict__ tiles, int n, int S, int ntx, int nx, int ny, int r,
                         const real* __restrict__ ftx, const real* __restrict__ fty, const real* __restrict__ ctx,
                         const real* __restrict__ cty, double inv_tau, const float* __restrict__ oscale,
                         float* __restrict__ y, float* __restrict__ mask, int* __restrict__ mcount) {
    const int So = S + 1, P = So * So;
    const size_t pfx = (size_t)r * ny * (nx + 1), pcx = (size_t)ny * (nx + 1);
    const size_t pfy = (size_t)(ny + 1) * r * nx, pcy = (size_t)(ny + 1) * nx;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n * P; k += gridDim.x * blockDim.x) {
        const int p = k / P, q = k % P, tile = tiles[p];
        const int gx = (tile % ntx) * S - 1 + q % So, gy = (tile / ntx) * S - 1 + q / So;
        float lab[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float msk[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (gx >= 0 && gy >= 0 && gx < nx && gy < ny) {
            if (gx + 1 < nx) {   // east face = x line I = gx + 1
                double f[3];
                for (int c = 0; c < 3; ++c) {
                    double sum = 0.0;
                    for (int j = 0; j < r; ++j) sum += (double)ftx[c * pfx + (size_t)(gy * r + j) * (nx + 1) + gx + 1];
                    f[c] = (sum / r - (double)ctx[c * pcx + (size_t)gy * (nx + 1) + gx + 1]) * inv_tau;
                }
                lab[0] = (float)f[0]; lab[1] = (float)f[1]; lab[2] = (float)f[2];
                msk[0] = msk[1] = msk[2] = 1.f;
            }
            if (gy + 1 < ny) {   // north face = y line J = gy + 1
                double f[3];
                for (int c = 0; c < 3; ++c) {
                    double sum = 0.0;
                    for (int i = 0; i < r; ++i) sum += (double)fty[c * pfy + (size_t)(gy + 1) * r * nx + gx * r + i];
                    f[c] = (sum / r - (double)cty[c * pcy + (size_t)(gy + 1) * nx + gx]) * inv_tau;
                }
                lab[3] = (float)f[0]; lab[4] = (float)f[2]; lab[5] = (float)f[1];   // world x, y momentum
                msk[3] = msk[4] = msk[5] = 1.f;
            }
        }
        int cnt = 0;
        for (int c = 0; c < 6; ++c) {
            y[(size_t)k * 6 + c] = lab[c] / oscale[c];
            mask[(size_t)k * 6 + c] = msk[c];
            cnt += msk[c] > 0.f;
        }
        if (cnt) atomicAdd(&mcount[p], cnt);
    }
}

// Minibatch: crops idx[b] of the data set into the network's input, label
// and mask buffers, BATCH_WG workgroups per crop; in pieces of 16 bytes (32 per
// input pixel) and 8 bytes (24 per output pixel), which every crop's start
// and size are multiples of.
constexpr int BATCH_WG = 8;
__global__ __launch_bounds__(256) void k_batch_copy(const int* __restrict__ idx, int So,
                                                    const unsigned short* __restrict__ X, const float* __restrict__ Y,
                                                    const float* __restrict__ M, unsigned short* __restrict__ x,
                                                    float* __restrict__ y, float* __restrict__ m) {
    const int Sin = So + 2 * HALO, b = blockIdx.x / BATCH_WG, t = blockIdx.x % BATCH_WG * 256 + threadIdx.x;
    const size_t src = idx[b];
    const int nx = Sin * Sin * 2, ny = So * So * 3;
    const uint4* const Xb = reinterpret_cast<const uint4*>(X) + src * nx;
    const uint2 *const Yb = reinterpret_cast<const uint2*>(Y) + src * ny, *const Mb = reinterpret_cast<const uint2*>(M) + src * ny;
    uint4* const xb = reinterpret_cast<uint4*>(x) + (size_t)b * nx;
    uint2 *const yb = reinterpret_cast<uint2*>(y) + (size_t)b * ny, *const mb = reinterpret_cast<uint2*>(m) + (size_t)b * ny;
    for (int k = t; k < nx || k < ny; k += BATCH_WG * 256) {
        if (k < nx) xb[k] = Xb[k];
        if (k < ny) { yb[k] = Yb[k]; mb[k] = Mb[k]; }
    }
}

// Host crops already rounded to FP32 (n, Sin, Sin, 6) into the network's bf16
// input with 16 channels, and labels and mask of a training batch (ny floats
// each, may be 0) beside them.
__global__ void k_crops_in(const float* __restrict__ hx, size_t npx, const float* __restrict__ hy,
                           const float* __restrict__ hm, size_t ny, unsigned short* __restrict__ x,
                           float* __restrict__ y, float* __restrict__ m) {
    const size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x, nt = (size_t)gridDim.x * blockDim.x;
    for (size_t p = t; p < npx; p += nt) {
        unsigned h[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            h[k] = to_bf16(hx[p * 6 + 2 * k]) | ((unsigned)to_bf16(hx[p * 6 + 2 * k + 1]) << 16);
        *reinterpret_cast<uint4*>(x + p * 16) = uint4{h[0], h[1], h[2], 0u};
        *reinterpret_cast<uint4*>(x + p * 16 + 8) = uint4{0u, 0u, 0u, 0u};
    }
    for (size_t k = t; k < ny; k += nt) { y[k] = hy[k]; m[k] = hm[k]; }
}

// Labels of the data set re-expressed in new output scales: y *= old / new.
__global__ void k_rescale(float* __restrict__ y, size_t n, const float* __restrict__ ratio) {
    for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x)
        y[k] *= ratio[k % 6];
}

}  // namespace lc
}  // namespace swe
