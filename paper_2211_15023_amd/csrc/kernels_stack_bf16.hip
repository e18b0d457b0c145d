// One whole stack of the IMPALA teacher in one kernel, bf16: conv3x3 (pad 1, no ReLU) -> max-pool 3x3 / 2 (pad 1) -> two
// residual blocks (ReLU - conv3x3 - ReLU - conv3x3 + skip).  The stack's input is read once and its output written once;
// every tensor in between stays in LDS.
//
// What bounds it: layer by layer the eleven launches of a stack moved the stream through memory nine times and fetched
// every window from LDS anew (nine or five 16-byte reads per lane and MFMA tile, as many LDS clocks as matrix clocks).
// Here a lane is a *column* of the image and walks down it: the fragments of an input row (three reads) serve the output
// rows above, at and below it, so a row of 16 pixels costs three reads and five (16 channels) or nine (32 channels) MFMAs
// per 16 output channels.  The three output rows in flight are three independent accumulator chains.  Measured at 1024
// states: the three stacks 66 / 63 / 31 us where the layer-by-layer kernels took 283 / 163 / 85 us; on another card 73-76 / 66-70 / 33-35 -> 69.6 /
// 63.4 / 31.5 with the order of bs_order and the input's chunks from a table.  What bounds it now: LDS in the first stack's blocks (3 200 of
// 4 000 clocks a phase), matrix cores in the others' (2 000 of 2 850), the pooling of all at 60-75 % of either.
//
//  * Lanes.  A workgroup of eight wavefronts owns G images.  The lanes of the blocks' tiles are (image, segment of rows,
//    column) triples: 3 x 42, 3 x 21 and 2 x 2 x 11 of them fill 126 of 128, 63 of 64 and 44 of 48 lanes.  32-channel
//    layers split the output channels over two wavefronts, so that a wavefront keeps the weights of all four block
//    convolutions (4 x 36 registers) for the whole kernel.
//  * LDS layout.  Planes of eight channels, [channel block][row][column][16 B]: the 16 lanes of a K group read 256
//    consecutive bytes, and planes a multiple of 256 bytes apart keep the four groups of a read off each other's banks.
//  * Convolution + pooling.  First stack: lanes are pooled pixels, the even and the odd column under each two sets of
//    accumulators (74 -> 71 us against seven pooled pixels per tile, which took twice the vector instructions per pixel); the odd
//    window is put together from the lane's even one and its neighbour's (read as well it was half of the phase's LDS clocks).
//    Others: lanes are convolution columns 14 t - 1 .. 14 t + 14 (seven pooled pixels).  The vertical
//    maximum runs over the rows as they are produced (row 2 py + 1 is kept for the next pooled row), the horizontal one
//    over the two neighbour lanes (DPP).  Rounding to bf16 is monotone, so it follows the maximum.
//  * The stream is kept un-rectified (the skip connection needs it) and rectified as fragments are read: one packed
//    16-bit integer maximum per dword, since a negative bf16 is a negative 16-bit integer (the NaN that the matrix cores
//    produce, 0xffc0, is one too and becomes 0 as in fmaxf).
//  * Inputs go from memory to LDS without passing through registers, a third of the next batch at the start of each of
//    three phases: loads into registers held their wavefront for 6 000 clocks of 34 000 in a full memory queue and storing
//    them took another 4 000 (second stack 80 -> 67 us, third 39 -> 32 us at 1024 states; the first with its odd windows 72.4 -> 69.6).
//
// Arithmetic: the planner's weight fragments, the bias in the accumulator and the K steps of every output in the planner's
// order, so results are bit-identical to the layer-by-layer kernels (conv_kernel.h), which the debug taps still run.  (The
// last K step of a 16-channel layer holds two chunks only; here they sit in the other half of the step, which adds the
// same products in the same order.)
#include <math.h>

#include <type_traits>

#include "conv_kernel.h"

namespace accerl {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));

struct BStackParams {
    const void* in;          // uint8 planes [B, 4, HIN, HIN] or bf16 [B, HIN, HIN, CI]
    const int32_t* rows;     // ROWS: observation i is row rows[i] of in
    char* out;               // bf16 [B, H, H, C]
    const v4i* w[5];         // 0: stack convolution, 1 / 2: first block's conv A / B, 3 / 4: second block's
    const float* bias[5];
    int64_t B;
};

constexpr int bs_up(int v, int a) { return (v + a - 1) / a * a; }

template <bool U8, int CI, int HIN, int C, int G_, int SEG_, int PSEG_>
struct BsShape {
    static constexpr int G = G_, SEG = SEG_, PSEG = PSEG_;
    static constexpr int NW = 8, THREADS = NW * 64;
    static constexpr int NH = C / 16;                          // wavefronts that share a tile, 16 output channels each
    static constexpr int TW = NW / NH;                         // tiles in work at a time
    static constexpr int H = (HIN - 1) / 2 + 1;                // pooled size
    // bordered tiles of the stream and of a block's inner tensor: planes of eight channels
    static constexpr int PB = H + 2, ROWB = PB * 16;
    static constexpr int R = (H + SEG - 1) / SEG;              // rows a lane walks
    static constexpr int PLANE = bs_up((PB + SEG * R - H) * ROWB, 256);
    static constexpr int TILE = C / 8 * PLANE;
    static constexpr int NCOL = G * SEG * H;
    // bordered input tile: channels-last pixels of 8 bytes (observations) or planes
    static constexpr int IPB = HIN + 2, IROW = IPB * (U8 ? 8 : 16);
    static constexpr int IPLANE = bs_up(IPB * IROW, 256);
    static constexpr int TILE_IN = U8 ? bs_up((HIN + 3) * IROW, 256) : CI / 8 * IPLANE;
    static constexpr int KS_C = U8 ? 2 : CI == 16 ? 5 : 9, KS_B = C == 16 ? 5 : 9;
    static constexpr int UNITS = HIN * HIN / 4;                // observations only
    static constexpr int PF = (UNITS + THREADS - 1) / THREADS;
    static constexpr int IMG_IN = U8 ? 4 * HIN * HIN : HIN * HIN * CI * 2;
    static constexpr int IMG = H * H * C * 2;
    // conv + pool items: column tiles of pooled pixels (14 of observations, else seven) x row segments x images
    static constexpr int CT = U8 ? (H + 13) / 14 : (H + 6) / 7, RP = (H + PSEG - 1) / PSEG, ITEMS = CT * PSEG * G;
    static constexpr int PAST = SEG * R - H;                   // rows that the last segment's lanes walk past the image
    // the inner tensor takes the place of the observation tile, which is dead once it has been pooled
    static constexpr bool OVER = U8;
    static constexpr int O_IN = G * TILE, O_M = O_IN;
    // where lanes that own no pooled pixel store (a branch around the store would end the compiler's view at every row)
    static constexpr int O_DUMP = O_M + (G * TILE > TILE_IN || !OVER ? G * TILE : TILE_IN);
    static constexpr int O_TAB = O_DUMP + RP * ROWB + 512;
    // inputs: an LDS array of their own, filled from memory without passing through registers (a load of 64 chunks each): the observation's
    // bytes as they are, or the planes and a table of where their chunks come from
    static constexpr int NLOAD = ((U8 ? IMG_IN : G * TILE_IN) / 16 + THREADS - 1) / THREADS, S_IN = U8 ? bs_up(IMG_IN, 1024) : NLOAD * THREADS * 16;
    static constexpr int LDS = O_TAB + (U8 ? 0 : NLOAD * THREADS * 4);    // dynamic; besides S_IN
    static_assert(PAST <= 1 && C % 16 == 0 && NCOL <= TW * 16 && (!U8 || (G == 1 && CI == 4)) && LDS + S_IN <= 160 * 1024, "shape");
};

__device__ __forceinline__ v4f bs_mfma(v4i a, v4i b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}
__device__ __forceinline__ v4i bs_relu(v4i x) {
    typedef short v8s __attribute__((ext_vector_type(8)));
    const v8s z = {0, 0, 0, 0, 0, 0, 0, 0};
    return __builtin_bit_cast(v4i, __builtin_elementwise_max(__builtin_bit_cast(v8s, x), z));
}
__device__ __forceinline__ v2i bs_pack(v4f v) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    return (v2i){__builtin_bit_cast(int, __builtin_convertvector((v2f){v[0], v[1]}, v2bf)),
                 __builtin_bit_cast(int, __builtin_convertvector((v2f){v[2], v[3]}, v2bf))};
}
__device__ __forceinline__ float bs_max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }
// max(v, v of both neighbours in the 16-lane row); the outermost lanes' results are not used
__device__ __forceinline__ float bs_max_neighbours(float v) {
    const int i = __float_as_int(v);
    return bs_max3(v, __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x111, 0xf, 0xf, false)),
                   __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x101, 0xf, 0xf, false)));
}

// 16 bytes a lane from the buffer to 1 KiB of LDS (the compiler's host pass does not know the builtin and would drop the kernel)
__device__ __forceinline__ void bs_load_lds(__amdgpu_buffer_rsrc_t src, char* lds, int off) {
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)lds, 16, off, 0, 0, 0);
#endif
}

// The fragments of one input row under a lane's 3-wide window.
// 16 channels (K steps of two pixels): f0 = pixels 0, 1; f1 = pixel 2 of the row above and pixel 0; f2 = pixels 1, 2.
// 32 channels (a pixel per step): f0, f1, f2 = pixels 0, 1, 2.
struct BsRow { v4i f[3]; };
template <int CIN>
__device__ __forceinline__ void bs_load(BsRow& r, const char* a, const char* m, int off) {
    r.f[0] = *(const v4i*)(a + off);
    r.f[1] = CIN == 16 ? *(const v4i*)(m + off) : *(const v4i*)(a + off + 16);
    r.f[2] = *(const v4i*)(a + off + (CIN == 16 ? 16 : 32));
}
// What an input row adds to the output rows whose last / middle / first window row it is: three chains, one product of each in turn.  A chain
// that is not wanted costs nothing once inlined.
template <int CIN>
__device__ __forceinline__ void bs_row(const v4i* w, const BsRow& r, v4f& bottom, v4f& mid, v4f& top) {
    if constexpr (CIN == 16) {
        bottom = bs_mfma(w[3], r.f[0], bottom);
        top = bs_mfma(w[0], r.f[0], top);
        mid = bs_mfma(w[1], r.f[1], mid);
        bottom = bs_mfma(w[4], r.f[2], bottom);
        mid = bs_mfma(w[2], r.f[2], mid);
    } else {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            bottom = bs_mfma(w[6 + q], r.f[q], bottom);
            mid = bs_mfma(w[3 + q], r.f[q], mid);
            top = bs_mfma(w[q], r.f[q], top);
        }
    }
}
// The order of a stretch of code without branches: R reads, then M times one product and V vector instructions.  Two wavefronts share a SIMD;
// left to itself the compiler puts a row's reads, products and vector instructions behind one another and waits between them.
template <int R, int M, int V>
__device__ __forceinline__ void bs_order() {
    __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
#pragma unroll
    for (int m = 0; m < M; ++m) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
    }
}

// ROWS: observations through the row list (as a test in the kernel it cost the others 0.5 us of 169 at 1024 states)
template <bool U8, int CI, int HIN, int C, int G, int SEG, int PSEG, bool ROWS>
__global__ __launch_bounds__(512, 2) void stack_bf16_kernel(const BStackParams p) {
    typedef BsShape<U8, CI, HIN, C, G, SEG, PSEG> S;
    constexpr int T = S::THREADS;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* tX = smem;                                     // G bordered tiles of the stream
    __shared__ __attribute__((aligned(16))) char s_in[S::S_IN];
    char* tin = S::OVER ? smem + S::O_IN : s_in;         // G bordered input tiles
    char* tM = smem + S::O_M;                            // G bordered tiles of a block's inner tensor
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int half = wave % S::NH, tile = wave / S::NH;  // which 16 output channels, which tile
    constexpr int NH = S::NH;

    // ---- staging of observations: unit u is one dword of each of the four planes
    auto commit = [&]() {
#pragma unroll
        for (int i = 0; i < S::PF; ++i) {
            const int u = tid + i * T;
            if (u >= S::UNITS) continue;
            constexpr int RU = HIN / 4;
            const int row = u / RU, cu = u - row * RU;
            int v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = *(const int*)(s_in + c * HIN * HIN + 4 * u);
            typedef float v2f __attribute__((ext_vector_type(2)));
            typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
            const float k255 = 1.0f / 255.0f;            // bf16(v / 255) = bf16(v * (1 / 255)): checked for all 256 values
            char* d = tin + (row + 1) * S::IROW + (1 + 4 * cu) * 8;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const v2f lo = {(float)((v[0] >> (8 * e)) & 0xff) * k255, (float)((v[1] >> (8 * e)) & 0xff) * k255};
                const v2f hi = {(float)((v[2] >> (8 * e)) & 0xff) * k255, (float)((v[3] >> (8 * e)) & 0xff) * k255};
                *(v2i*)(d + 8 * e) = (v2i){__builtin_bit_cast(int, __builtin_convertvector(lo, v2bf)),
                                           __builtin_bit_cast(int, __builtin_convertvector(hi, v2bf))};
            }
        }
        for (int i = tid; i < 3 * S::IPB; i += T) {      // the border of the observation tile: three rows, two columns
            const int rr = i / S::IPB;
            *(v2i*)(tin + (rr ? HIN + rr : 0) * S::IROW + (i - rr * S::IPB) * 8) = (v2i){0, 0};
        }
        for (int i = tid; i < 2 * HIN; i += T) *(v2i*)(tin + (1 + (i >> 1)) * S::IROW + (i & 1) * (HIN + 1) * 8) = (v2i){0, 0};
    };
    // ---- memory to s_in directly.  Observations: chunk by chunk (into registers, with their 16 loads in the last phase, they held it for
    //      2 300 clocks of 5 900).  bf16: chunk i * T + tid of the planes comes from tab[i * T + tid] of the batch; those of borders and padding, and
    //      of images past the batch, are out of the buffer's range: zeros.  (Worked out for every load, a third of the loads cost their
    //      phase 1 100 clocks of 4 000.)
    int* tab = (int*)(smem + S::O_TAB);
    auto fetch = [&](int64_t batch, int i0, int i1) {
        const int64_t b0 = batch * G;
        const auto src = __builtin_amdgcn_make_buffer_rsrc((char*)p.in + (ROWS ? (int64_t)p.rows[b0] : b0) * (int64_t)S::IMG_IN, 0,
                                                           (int)min(p.B - b0, (int64_t)G) * S::IMG_IN, 0x00027000);
#pragma unroll
        for (int i = i0; i < i1; ++i) {
            if (i >= S::NLOAD) continue;
            if constexpr (!U8) bs_load_lds(src, s_in + (wave + i * S::NW) * 1024, tab[i * T + tid]);
            else if ((i + 1) * T * 16 <= S::S_IN || (wave + i * S::NW) * 1024 < S::S_IN) bs_load_lds(src, s_in + (wave + i * S::NW) * 1024, (i * T + tid) * 16);
        }
    };
    if constexpr (!U8) {
#pragma unroll
        for (int i = 0; i < S::NLOAD; ++i) {
            const int q = tid + i * T;
            const int im = q / (S::TILE_IN / 16), r1 = q - im * (S::TILE_IN / 16), cb = r1 / (S::IPLANE / 16), r2 = r1 - cb * (S::IPLANE / 16);
            const int row = r2 / S::IPB, col = r2 - row * S::IPB;
            const bool pixel = im < G && row >= 1 && row <= HIN && col >= 1 && col <= HIN;
            tab[q] = pixel ? im * S::IMG_IN + ((row - 1) * HIN + col - 1) * (CI * 2) + cb * 16 : 0x7fffff00;
            if (!pixel) ((v4i*)s_in)[q] = (v4i){0, 0, 0, 0};
        }
    }

    const int64_t n_batch = (p.B + G - 1) / G;
    int64_t batch = blockIdx.x;
    if (batch < n_batch) {
        fetch(batch, 0, S::NLOAD);
    }

    // ---- weights of all five convolutions, in registers for the whole kernel
    v4i wC[S::KS_C], wA1[S::KS_B], wB1[S::KS_B], wA2[S::KS_B], wB2[S::KS_B];
    v4f bias[5];
    {
        auto frag = [&](int cv, int st, int ks) -> v4i {
            if (ks == 5 && st == 4) {                    // the two chunks of the last step in the upper half (bs_row multiplies it with pixels 1, 2)
                const v4i v = p.w[cv][(st * NH + half) * 64 + (lane & 31)];
                return g >= 2 ? v : (v4i){0, 0, 0, 0};
            }
            return p.w[cv][(st * NH + half) * 64 + lane];
        };
#pragma unroll
        for (int st = 0; st < S::KS_C; ++st) wC[st] = frag(0, st, S::KS_C);
#pragma unroll
        for (int st = 0; st < S::KS_B; ++st) {
            wA1[st] = frag(1, st, S::KS_B);
            wB1[st] = frag(2, st, S::KS_B);
            wA2[st] = frag(3, st, S::KS_B);
            wB2[st] = frag(4, st, S::KS_B);
        }
#pragma unroll
        for (int cv = 0; cv < 5; ++cv) bias[cv] = *(const v4f*)(p.bias[cv] + 4 * NH * g + 4 * half);
    }
    for (int i = tid; i < S::O_TAB / 16; i += T) ((v4i*)smem)[i] = (v4i){0, 0, 0, 0};

    // ---- this lane's column of the blocks' tiles
    const int n = tile * 16 + j, nc = min(n, S::NCOL - 1);
    const int img = nc / (SEG * S::H), seg = (nc - img * SEG * S::H) / S::H, col = nc - (img * SEG + seg) * S::H;
    const int row0 = seg * S::R;
    const int pos = img * S::TILE + row0 * S::ROWB + col * 16;
    const int offA = pos + (C == 16 ? (g & 1) * S::PLANE + (g >> 1) * 16 : g * S::PLANE);
    const int offM = pos + (g & 1) * S::PLANE + (g < 2 ? 32 - S::ROWB : 0);       // 16 channels only
    const int own = pos + S::ROWB + 16 + (C == 16 ? (g >> 1) * S::PLANE + (g & 1) * 8 : g * S::PLANE + half * 8);
    const int past = S::PAST && seg == SEG - 1 ? S::ROWB : 0;
    if constexpr (U8) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // (see the loop's end)
    __syncthreads();

    for (; batch < n_batch; batch += gridDim.x) {
        if constexpr (U8) commit();
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wavefront's part of the input is in LDS
        __syncthreads();
        const int64_t b0 = batch * G;
        const int gc = (int)((p.B - b0 < G) ? (p.B - b0) : G);

        // ---- stack convolution + max-pool -> the stream's tile
        for (int it = tile; it < S::ITEMS; it += S::TW) {
            const int im = it / (S::CT * PSEG), ps = (it - im * S::CT * PSEG) % PSEG, ct = (it - im * S::CT * PSEG) / PSEG;
            const int p0 = min(ps * S::RP, S::H - S::RP);        // segments may overlap: the same bytes twice
            auto dst_of = [&](int px, bool ok) {
                return !ok ? smem + S::O_DUMP + 8 * lane : tX + im * S::TILE + (p0 + 1) * S::ROWB + (px + 1) * 16 + (C == 16 ? (g >> 1) * S::PLANE + (g & 1) * 8 : g * S::PLANE + half * 8);
            };
            const v4f none = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if constexpr (U8) {
                // Lanes are pooled pixels 14 ct .. 14 ct + 15 with the even and the odd column (E, O) as two sets of accumulators; the
                // left neighbour's O completes the window (the first pixel of all needs none), the right one's fragment is the second
                // half of the odd column's: the first and the last lane only serve their neighbours.
                const int px = 14 * ct + j, pc = min(px, S::H);
                char* dst = dst_of(px, (ct == 0 || j >= 1) && j <= 14 && px < S::H);
                // window rows y, y + 1 in the two halves of a fragment: F(y) is step 0 of conv row y and step 1 of row y - 2
                const char* a = tin + (2 * p0 + (g >> 1)) * S::IROW + 2 * pc * 8 + (g & 1) * 16;
                auto even = [&](int row) { return *(const v4i*)(a + row * S::IROW); };
                auto odd = [&](v4i e) {
                    return (v4i){e[2], e[3], __builtin_amdgcn_update_dpp(e[2], e[0], 0x101, 0xf, 0xf, false), __builtin_amdgcn_update_dpp(e[3], e[1], 0x101, 0xf, 0xf, false)};
                };
                static_assert(S::IROW % 16 == 0 && HIN % 2 == 0, "whole chunks under even columns");
                auto conv = [&](v4i lo, v4i hi) { return bs_mfma(wC[1], hi, bs_mfma(wC[0], lo, bias[0])); };
                v4i e0 = even(0), e1 = even(1), o0 = odd(e0), o1 = odd(e1);
                v4f carryE = none, carryO = none;
                if (p0 > 0) { carryE = conv(even(-1), e1); carryO = conv(odd(even(-1)), o1); }
                v4i e2 = even(2), e3 = even(3), o2 = odd(e2), o3 = odd(e3);
                v4i eN = even(4), fN = even(5);
                v4f cE0 = conv(e0, e2), cO0 = conv(o0, o2), cE1 = conv(e1, e3), cO1 = conv(o1, o3);
#pragma unroll
                for (int k = 0; k < S::RP; ++k) {
                    v4f mO, mE;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        mO[r] = bs_max3(carryO[r], cO0[r], cO1[r]);
                        mE[r] = bs_max3(carryE[r], cE0[r], cE1[r]);
                    }
                    carryE = cE1; carryO = cO1;
                    if (k + 1 < S::RP) {                  // the next row's products go between this one's maxima
                        e0 = e2; e1 = e3; o0 = o2; o1 = o3;
                        e2 = eN; e3 = fN;
                        if (k + 2 < S::RP) { eN = even(2 * k + 6); fN = even(2 * k + 7); }
                        o2 = odd(e2); o3 = odd(e3);
                        cE0 = conv(e0, e2); cE1 = conv(e1, e3); cO0 = conv(o0, o2); cO1 = conv(o1, o3);
                    }
                    v4f m;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int i = __float_as_int(mO[r]);
                        m[r] = bs_max3(mE[r], mO[r], __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x111, 0xf, 0xf, false)));
                    }
                    *(v2i*)(dst + k * S::ROWB) = bs_pack(m);
                    if (k + 1 < S::RP) bs_order<2, 8, 3>();
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                const int x = min(max(14 * ct - 1 + j, 0), HIN - 1);  // columns outside repeat the outermost one
                const int px = 7 * ct + (j >> 1);
                char* dst = dst_of(px, (j & 1) && j < 14 && px < S::H);
                auto store = [&](int k, v4f v) {
                    v4f m;
#pragma unroll
                    for (int r = 0; r < 4; ++r) m[r] = bs_max_neighbours(v[r]);
                    *(v2i*)(dst + k * S::ROWB) = bs_pack(m);
                };
                v4f carry = none;
                const int base = im * S::TILE_IN + 2 * p0 * S::IROW + x * 16;
                const char* a = tin + base + (CI == 16 ? (g & 1) * S::IPLANE + (g >> 1) * 16 : g * S::IPLANE);
                const char* m = tin + base + (g & 1) * S::IPLANE + (g < 2 ? 32 - S::IROW : 0);
                BsRow r0, r1;                             // input rows 2 p0, 2 p0 + 1
                bs_load<CI>(r1, a, m, S::IROW);
                v4f a1, a2, unused = none;
                if (p0 > 0) {                             // conv row 2 p0 - 1, kept for the first pooled row
                    BsRow rm;
                    bs_load<CI>(rm, a, a, -S::IROW);      // (its f1 is not used with 16 channels)
                    bs_load<CI>(r0, a, m, 0);
                    carry = bias[0];
                    bs_row<CI>(wC, rm, unused, unused, carry);
                    a2 = a1 = bias[0];
                    bs_row<CI>(wC, r0, unused, carry, a2);
                    bs_row<CI>(wC, r1, carry, a2, a1);
                } else {
                    bs_load<CI>(r0, a, a, 0);
                    a2 = a1 = bias[0];
                    bs_row<CI>(wC, r0, unused, unused, a2);
                    bs_row<CI>(wC, r1, unused, a2, a1);
                }
                constexpr int NM = CI == 16 ? 5 : 9;
                BsRow r2, r3;
                bs_load<CI>(r2, a, m, 2 * S::IROW);
                v4f v = none;
#pragma unroll
                for (int k = 0; k < S::RP; ++k) {
                    const bool low = (HIN & 1) == 0 || k + 1 < S::RP || p0 + k < S::H - 1;   // conv row 2 py + 1 exists
                    // conv row 2 py is complete with row 2, the next two are under way; the maximum of the row above follows the products
                    if (low) bs_load<CI>(r3, a, m, (2 * k + 3) * S::IROW);
                    v4f c0 = a2, c1 = a1, top = bias[0];
                    bs_row<CI>(wC, r2, c0, c1, top);
                    if (k > 0) store(k - 1, v);
                    if (low) bs_order<3, NM, CI == 16 ? 5 : 3>();
                    __builtin_amdgcn_sched_barrier(0);
                    if (k + 1 < S::RP) bs_load<CI>(r2, a, m, (2 * k + 4) * S::IROW);
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = fmaxf(carry[r], c0[r]);
                    if (low) {
                        a2 = top; a1 = bias[0];
                        bs_row<CI>(wC, r3, c1, a2, a1);
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], c1[r]);
                        carry = c1;
                    }
                    if (k + 1 < S::RP) bs_order<3, NM, 1>();
                    __builtin_amdgcn_sched_barrier(0);
                }
                store(S::RP - 1, v);
            }
        }
        __syncthreads();
        if constexpr (S::OVER) {                          // the inner tensor's border, where the observation tile was
            for (int i = tid; i < C / 8 * (2 * S::PB + 2 * S::H); i += T) {
                const int pl = i / (2 * S::PB + 2 * S::H), q = i - pl * (2 * S::PB + 2 * S::H);
                int at;
                if (q < 2 * S::PB) at = (q < S::PB ? q : (S::H + 1) * S::PB + q - S::PB);
                else at = (1 + ((q - 2 * S::PB) >> 1)) * S::PB + (q & 1) * (S::H + 1);
                *(v4i*)(tM + pl * S::PLANE + at * 16) = (v4i){0, 0, 0, 0};
            }
        }

        // ---- one block convolution: walk down this lane's column; done(k, acc) takes output row k, one row late, and before(k) what it will need
        auto walk = [&](const char* src, const v4i* w, v4f b, auto relu, auto&& before, auto&& done) {
            constexpr bool RELU = decltype(relu)::value;
            constexpr int NM = C == 16 ? 5 : 9;
            const char* a = src + offA;
            const char* m = src + offM;
            BsRow cur, nxt;
            auto rect = [&](BsRow& r) {
                if constexpr (RELU) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) r.f[q] = bs_relu(r.f[q]);
                }
            };
            bs_load<C>(cur, a, a, 0);                     // (f1 of the first row is not used with 16 channels)
            bs_load<C>(nxt, a, m, S::ROWB);
            rect(cur);
            v4f a2 = b, a1 = b, out = b, unused = b;
            bs_row<C>(w, cur, unused, unused, a1);
#pragma unroll
            for (int i = 1; i < S::R + 2; ++i) {
                cur = nxt;
                if (i + 1 < S::R + 2) bs_load<C>(nxt, a, m, (i + 1) * S::ROWB);
                if (i >= 2) before(i - 2);
                rect(cur);
                // (chains of rows above the first and past the last are not used)
                v4f o = a2, mid = a1, top = b;
                bs_row<C>(w, cur, o, mid, top);
                if (i >= 3) done(i - 3, out);
                if (i >= 3 && i < S::R) {
                    if constexpr (RELU) __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
                    bs_order<RELU ? 3 : 4, NM, C == 16 ? (RELU ? 3 : 2) : (RELU ? 2 : 1)>();
                }
                __builtin_amdgcn_sched_barrier(0);
                out = o; a2 = mid; a1 = top;
            }
            done(S::R - 1, out);
        };
        // Lanes past the last column repeat it, those of images past the batch work on what is there: no predicates.  The row that the last
        // segment's lanes walk past the image goes to the row behind the border, which meets no pixel of the image.
        auto at = [&](int k) { return own + (k + 1 == S::R ? past : 0) + k * S::ROWB; };
        auto conv_a = [&](const v4i* w, v4f b) {          // inner tensor = relu(conv(relu(stream)))
            if (tile * 16 >= S::NCOL) return;
            walk(tX, w, b, std::true_type{}, [](int) {}, [&](int k, v4f acc) {
                typedef short v4s __attribute__((ext_vector_type(4)));
                const v4s q = __builtin_elementwise_max(__builtin_bit_cast(v4s, bs_pack(acc)), (v4s){0, 0, 0, 0});
                *(v2i*)(tM + at(k)) = __builtin_bit_cast(v2i, q);
            });
        };
        auto conv_b = [&](const v4i* w, v4f b, auto last) {   // stream += conv(inner tensor), in place or to memory
            constexpr bool LAST = decltype(last)::value;
            if (tile * 16 >= S::NCOL) return;
            const int offp = ((img * S::H + row0) * S::H + col) * (C * 2) + (C == 16 ? 8 * g : 16 * g + 8 * half);
            char* outp = p.out + b0 * (int64_t)S::IMG + (uint32_t)offp;
            // (the buffer ends with the batch's last image: what is stored behind it is dropped)
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(p.out + b0 * (int64_t)S::IMG, 0, gc * S::IMG, 0x00027000);
            v2i x[2];
            walk(tM, w, b, std::false_type{}, [&](int k) { x[k & 1] = *(const v2i*)(tX + own + k * S::ROWB); }, [&](int k, v4f acc) {
                const v2i q = x[k & 1];
                const v4f y = {bf2f((uint32_t)q[0] & 0xffffu) + acc[0], __int_as_float(q[0] & (int)0xffff0000) + acc[1],
                               bf2f((uint32_t)q[1] & 0xffffu) + acc[2], __int_as_float(q[1] & (int)0xffff0000) + acc[3]};
                if constexpr (!LAST) *(v2i*)(tX + at(k)) = bs_pack(y);
                else if constexpr (G == 1 && S::PAST == 0) *(v2i*)(outp + k * S::H * C * 2) = bs_pack(y);
                else {
                    typedef unsigned v2u __attribute__((ext_vector_type(2)));
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, bs_pack(y)), rsrc, k + 1 == S::R && past ? 0x7fffff00 : offp, k * S::H * C * 2, 0);
                }
            });
        };
        // the next batch's input, a third of the loads at a time: the memory queue of a compute unit holds a wavefront that
        // issues into it when it is full
        const int64_t next = batch + gridDim.x;
        constexpr int N3 = (S::NLOAD + 2) / 3;
        if (next < n_batch) fetch(next, 0, N3);
        conv_a(wA1, bias[1]);
        __syncthreads();
        if (next < n_batch) fetch(next, N3, 2 * N3);
        conv_b(wB1, bias[2], std::false_type{});
        __syncthreads();
        if (next < n_batch) fetch(next, 2 * N3, S::NLOAD);
        conv_a(wA2, bias[3]);
        __syncthreads();
        conv_b(wB2, bias[4], std::true_type{});
        // the observation tile takes the inner tensor's place, and its bytes were fetched by all wavefronts; otherwise the barrier behind the
        // next commit is enough
        if constexpr (S::OVER) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
    }
}

// the five convolutions of a stack as the planner laid them out
template <bool U8, int CI, int HIN, int C, int G, int SEG, int PSEG>
bool bs_shape_ok(const ConvParams& c, const ConvParams& a1, const ConvParams& b1, const ConvParams& a2, const ConvParams& b2) {
    typedef BsShape<U8, CI, HIN, C, G, SEG, PSEG> S;
    if (c.H != HIN || c.W != HIN || c.Cs_in != CI || c.Cin_real != CI || c.Ho != HIN || c.Wo != HIN || c.Cs_out != C) return false;
    if (c.k != 3 || c.s != 1 || c.pad != 1 || c.sx != 1 || c.k_steps != S::KS_C || (c.src_u8 != 0) != U8 || c.relu || c.relu_in) return false;
    for (const ConvParams* b : {&a1, &b1, &a2, &b2}) {
        if (b->H != S::H || b->W != S::H || b->Cin_real != C || b->Cs_in != C || b->Ho != S::H || b->Wo != S::H || b->Cs_out != C) return false;
        if (b->k != 3 || b->s != 1 || b->pad != 1 || b->sx != 1 || b->k_steps != S::KS_B || b->src_u8 || b->pool || b->out_frag) return false;
    }
    return a1.relu_in && a1.relu && !b1.relu_in && !b1.relu && a2.relu_in && a2.relu && !b2.relu_in && !b2.relu;
}

template <bool U8, int CI, int HIN, int C, int G, int SEG, int PSEG, bool ROWS = false>
hipError_t bs_go(const BStackParams& p, hipStream_t s) {
    if constexpr (U8 && !ROWS) { if (p.rows) return bs_go<U8, CI, HIN, C, G, SEG, PSEG, true>(p, s); }
    typedef BsShape<U8, CI, HIN, C, G, SEG, PSEG> S;
    auto kfn = stack_bf16_kernel<U8, CI, HIN, C, G, SEG, PSEG, ROWS>;
    static const hipError_t attr = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
    if (attr != hipSuccess) return attr;
    // one workgroup per compute unit (LDS and registers), striding over the batches in even rounds
    const int64_t batches = (p.B + G - 1) / G, cap = conv_num_cus();
    const int64_t rounds = (batches + cap - 1) / cap;
    kfn<<<dim3((unsigned)((batches + rounds - 1) / rounds)), dim3(S::THREADS), S::LDS, s>>>(p);
    return hipGetLastError();
}

}  // namespace

// (uint8 source, input channels, input size, channels, images per batch, row segments of the blocks' and of the pool's lanes)
#define ACCERL_BSTACK_SHAPES(X) X(true, 4, 84, 16, 1, 3, 5) X(false, 16, 42, 32, 1, 3, 4) X(false, 32, 21, 32, 2, 2, 1)

bool stack_bf16_supported(const ConvParams& c, const ConvParams& a1, const ConvParams& b1, const ConvParams& a2, const ConvParams& b2) {
#define X(U8, CI, HIN, C, G, SEG, PSEG) if (bs_shape_ok<U8, CI, HIN, C, G, SEG, PSEG>(c, a1, b1, a2, b2)) return true;
    ACCERL_BSTACK_SHAPES(X)
#undef X
    return false;
}

hipError_t launch_stack_bf16(const ConvParams& c, const ConvParams& a1, const ConvParams& b1, const ConvParams& a2, const ConvParams& b2, hipStream_t s) {
    if (c.B <= 0) return hipSuccess;
    BStackParams p;
    p.in = c.in; p.rows = c.rows; p.out = (char*)b2.out;
    const ConvParams* cv[5] = {&c, &a1, &b1, &a2, &b2};
    for (int i = 0; i < 5; ++i) { p.w[i] = (const v4i*)cv[i]->wfrag; p.bias[i] = (const float*)cv[i]->bias; }
    p.B = c.B;
#define X(U8, CI, HIN, C, G, SEG, PSEG) if (bs_shape_ok<U8, CI, HIN, C, G, SEG, PSEG>(c, a1, b1, a2, b2)) return bs_go<U8, CI, HIN, C, G, SEG, PSEG>(p, s);
    ACCERL_BSTACK_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace accerl
