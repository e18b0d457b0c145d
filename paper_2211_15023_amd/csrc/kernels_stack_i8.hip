// One whole stack of the IMPALA-style student in one kernel: conv3x3 (pad 1, no ReLU) -> max-pool 3x3 / 2 (pad 1)
// -> two residual blocks (ReLU - conv3x3 - ReLU - conv3x3 + skip), all int8.  Layer by layer (even with the pool and
// each block fused) a stack moves its stream through memory nine times; here the observation (or the stack before)
// is read once and the stack's output written once, and every tensor in between lives in LDS or in registers.
//
// What bounds these layers is not the matrix cores but the vector instructions around them (requantization, pooling,
// addressing), two clocks of a SIMD each (32-bit additions, subtractions, products and logic on vector registers) or four
// (conversions, minima and maxima, shifts, byte permutes, anything with a scalar register).  The kernel is therefore
// organised to issue few of them:
//
//  * Lanes are columns of the image and walk down it: a fragment read from LDS serves every output row whose window holds
//    it, and a row's address is a per-lane constant plus an immediate.  (Tiles of 16 pixels in raster order read every
//    window anew and looked each one up in a table: 9 instead of 2 further instructions beside the 12 of a requantized
//    ReLU row of four channels, and two to three times the LDS reads.)  The lanes of a workgroup's wavefronts are (image,
//    segment of rows, column) triples: 6 x 21 of 128 (a column is two pixels of 8 channels), 3 x 21 of 64, 5 x 11 of 64.
//    Where the columns do not fill the lanes, the last ones repeat a column of the same wavefront: no predicates.
//  * Block convolutions, 16 channels: a K step is one window row (three pixels; the fourth lane group reads the zeros of
//    the left border), so the fragment of an input row is multiplied with the weights of its three places in a window.
//    8 channels (two adjacent pixels fill the 16 MFMA rows): a fragment is two rows of four pixels, and two fragments are
//    the four rows that two output rows need, multiplied with the weights of the upper and of the lower one: one read
//    and four MFMAs per two rows.
//  * Convolution + pooling without storing the convolution.  Requantization is monotone per channel, so pooling the int32
//    accumulators first and requantizing the maxima gives the same bytes with a quarter of the requantizations.  A lane is
//    a pooled pixel; the four rows of four pixels under it give both conv rows 2py, 2py+1 of its even and odd columns (E =
//    2px, O = 2px+1).  The vertical maximum takes the lower conv row of the pooled row above (8-channel layers walk down
//    strips for it, with the next windows read before the results are stored: two reads and four MFMAs per pair of rows in place of
//    three and five, 340 -> 328 us for the first stack with the observations by buffer loads), the horizontal one is
//    max(E, O, O of the pixel to the left), the last term one DPP row shift; a tile's first lane only serves its neighbour
//    (tiles advance by 15 pixels).  The first column needs no left neighbour: 16-channel layers, whose tiles hold several
//    runs of columns, put a dummy in front of each run.  Rows and columns outside the image are replaced by their nearest
//    neighbour inside, which is part of the same window, so no -infinity is needed.  8-channel layers: the MFMA rows are
//    ordered so that a lane holds E and O of two channels (E and O in the two halves of a wavefront took a swap and two
//    more maxima per register: 340 -> 320 us for the first stack).
//  * The pooled stream goes to LDS twice: max(x, 0) where the first block's conv A reads it, and x itself where the inner
//    tensor will be; the lanes that own its pixels take it into registers (a dword per row) before they write the inner
//    tensor there.  From then on the skip connection stays in registers.  max(x, 0) of four packed bytes costs two
//    instructions: v_perm_b32 spreads the signs of the 16-bit halves the bytes are packed from.
//  * The weights of the block convolutions are read from LDS at the start of each phase (all of them in registers held
//    the wavefronts at 188, two to a SIMD: 435 -> 345 us for the first stack at 128), a few stay in registers where LDS
//    is what limits the workgroups.
//  * the next batch's input bytes are requested at the start of the current batch's last phase and land while it runs.
//
// Measured at 16384 states (kernel traces): 429 / 270 / 95 us with tiles in raster order, now 295-309 / 165-173 / 67-69 (two cards).
// Vector instructions at four clocks each 85 / 80 / 61 % of the clocks (an overstatement, see above), LDS pipe 60 / 49 / 40 %, matrix
// cores 29 / 46 / 39 %.  What the clocks go to is not settled by that: the first stack, 330 us, took 270 without its requantizations,
// 270 without its products and 228 without either, 325 without the LDS reads of the walks and 326 without barriers.  The 228 -- pooling
// maxima, the skip connection's unpacking, staging, LDS stores, addresses -- have not been taken apart.
//
// Arithmetic and constants are those of the layer-by-layer kernels (conv_kernel.h), so results are bit-identical; the debug
// taps still run that path.  Network: the benchmark's IMPALA configuration (three such stacks).
#include <stdlib.h>

#include <type_traits>

#include "conv_kernel.h"

namespace accerl {

namespace {

struct StackParams {
    const void* in;          // uint8 planes [B, 4, HIN, HIN] or int8 [B, HIN, HIN, CI]
    const int32_t* rows;     // observation i is row rows[i] of in (NULL = row i; an instance of its own: 604.6 for 604.9 us at 16384 states)
    int8_t* out;             // [B, H, H, C]
    const v4i* w[5];         // 0: stack convolution, 1 / 2: first block's conv A / B, 3 / 4: second block's
    const int* bias[5];
    const float* mult[5];
    float r1, r2;            // scale of a block's input over the scale of its output
    int64_t B;
    int units;               // compute units: workgroup b of the resident ones is number b / units on its unit
};

constexpr int st_up16(int v) { return (v + 15) / 16 * 16; }

template <bool U8, int CI, int HIN, int C, int G_, int SEG_, int PSEG_, int NW_, int WL_>
struct StShape {
    static constexpr int G = G_, SEG = SEG_, PSEG = PSEG_, WL = WL_;
    static constexpr int NW = NW_, THREADS = NW * 64;         // wavefronts per workgroup
    static constexpr int P = 16 / C;                          // output pixels per MFMA column (2 for 8 channels)
    // input tile: one pixel of border on every side
    static constexpr int PITCH_IN = st_up16((HIN + 2) * CI);
    static constexpr int TILE_IN = (HIN + 2) * PITCH_IN;
    static constexpr int UPR_IN = U8 ? HIN / 4 : HIN * CI / 16; // staging units per image row
    static constexpr int UNITS_IN = HIN * UPR_IN;
    static constexpr int IMG_IN = U8 ? 4 * HIN * HIN : HIN * HIN * CI;
    static constexpr int PF = (G * UNITS_IN + THREADS - 1) / THREADS;
    // the observation's unit that lane tid stages i-th; one that does not exist re-reads the last (three of a lane's four always exist)
    static constexpr int unit(int tid, int i) { return (i + 1) * THREADS <= UNITS_IN || tid + i * THREADS < UNITS_IN ? tid + i * THREADS : UNITS_IN - 1; }
    static constexpr int CPR_C = ((3 + P - 1) * CI + 15) / 16;  // 16-byte chunks per kernel row of the planner's fragments
    static constexpr int KS_C = (3 * CPR_C + 3) / 4;
    // pooled stream
    static constexpr int H = (HIN - 1) / 2 + 1;
    static constexpr int RP = (H + PSEG - 1) / PSEG;            // pooled rows a lane walks
    static constexpr int SLOTS = G * PSEG * (H + 1) - 1;        // a dummy slot in front of every column run but the first
    static constexpr int NT1 = SLOTS <= 16 ? 1 : 1 + (SLOTS - 16 + 14) / 15;
    // residual blocks
    static constexpr int WP = H / P;                           // columns per image row
    static constexpr int R = H / SEG;                          // rows a lane walks
    static constexpr int NCOL = G * SEG * WP;                  // lanes
    static constexpr int IMG = H * H * C;
    static constexpr int PITCH_B = st_up16((H + 3) * C);       // the pixel behind the border takes what the pooling's spare lanes write
    // a row behind the border is read (and meets zero weights): the second of a pair
    static constexpr int TILE_B = (H + 2 + (P == 2 ? 1 : 0)) * PITCH_B;
    static constexpr int CPR_B = ((3 + P - 1) * C + 15) / 16;
    static constexpr int KS_B = (3 * CPR_B + 3) / 4;
    static constexpr int NWB = P == 2 ? 4 : 3;                 // fragments of a block convolution
    static constexpr int WB = P == 2 ? 4096 : 9 * 256;         // their bytes in LDS (three lane groups of 16-channel layers)
    static constexpr int NWP = P == 2 ? 2 : CI == 8 ? 8 : 6;   // fragments of the stack convolution
    // The products of a row are issued between the vector instructions of the row above, their fragments read before that.  Left to itself
    // the compiler keeps every read behind the stores of the row above and waits for it and then for the products.  For the third stack,
    // whose LDS leaves a SIMD two wavefronts (1024 states 12.3 -> 11.1 us, 4096 29.5 -> 28.3, 16384 79.3 -> 75.6; the blocks alone 11.4, 28.8,
    // 77.5); the others' four cover each other and have no registers for it (first 333 / 333, second 188 / 190 with spills).
    static constexpr bool AHEAD = CI == 16;
    // LDS layout (bytes)
    static constexpr int O_TX = st_up16(G * TILE_IN + 64);
    static constexpr int O_TM = O_TX + G * TILE_B;
    static constexpr int O_W = O_TM + G * TILE_B;              // weight fragments of the first WL block convolutions
    static constexpr int O_CST = O_W + WL * WB;
    static constexpr int LDS = O_CST + 5 * 2 * 16 * 4;
    static_assert(H % P == 0 && (U8 ? (HIN % 4 == 0 && CI == 4 && G == 1) : (HIN * CI) % 16 == 0), "shape");
    static_assert(NCOL <= NW * 16 && NT1 <= NW * (P == 2 ? 99 : 1), "one tile of columns per wavefront");
    static_assert(P == 1 || (G == 1 && KS_C == 1 && KS_B == 2 && H % 2 == 0 && HIN % 2 == 0), "8-channel layers: one image, even sizes");
    static_assert(P == 2 || (KS_B == 3 && (CI == 8 || CI == 16) && (CI == 16 || HIN % 2 == 0)), "16-channel layers");
    static_assert(LDS <= 160 * 1024 && WL <= 4 && SEG * R == H && (HIN % 2 == 0 || PSEG == 1), "LDS, rows");
    static_assert(NCOL > NW * 16 - 16, "every wavefront owns a column");
};
// The loads of an observation's planes have the plane as their scalar offset, which a buffer's range check may leave out: a lane's offset
// stays inside a plane by itself.
template <class S>
constexpr bool st_units_in_plane(int plane) {
    for (int i = 0; i < S::PF; ++i)
        for (int tid = 0; tid < S::THREADS; ++tid)
            if (4 * S::unit(tid, i) + 4 > plane) return false;
    return true;
}

// v[r] = max(v[r], v[r] of the lane to its left in the same 16-lane row); lane 0 of a row keeps its value: a DPP lane without
// a source is not written and keeps the destination's old value.  (The two idle cycles a DPP read needs after the vector
// instruction that wrote its source are spelled out: the compiler does not look inside the statement.)
__device__ __forceinline__ void max_with_left(int (&v)[4]) {
    asm("s_nop 1\n\tv_max_i32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\tv_max_i32_dpp %1, %1, %1 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_max_i32_dpp %2, %2, %2 row_shr:1 row_mask:0xf bank_mask:0xf\n\tv_max_i32_dpp %3, %3, %3 row_shr:1 row_mask:0xf bank_mask:0xf"
        : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
}

__device__ __forceinline__ v4i st_mfma(v4i a, v4i b, v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0); }

// Four clamped results (rne_clamp127: the low 16 bits are the value as int16) -> their bytes, and max(., 0) of the bytes:
// the two halves as 16-bit pairs, whose sign bits v_perm_b32 spreads over a byte each.
struct StBytes { uint32_t raw, pos; };
__device__ __forceinline__ StBytes st_pack(const int (&q)[4]) {
    const uint32_t lo = __builtin_amdgcn_perm((uint32_t)q[1], (uint32_t)q[0], 0x05040100u);
    const uint32_t hi = __builtin_amdgcn_perm((uint32_t)q[3], (uint32_t)q[2], 0x05040100u);
    const uint32_t raw = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
    const uint32_t neg = __builtin_amdgcn_perm(hi, lo, 0x0b0a0908u);
    return {raw, raw & ~neg};
}

// BITS: the sums are small enough to be read as floats without a conversion (half the clocks of a subtraction): those of the
// blocks' first convolutions start at bias + 0x4B000000 (see requant_relu4_p23), the others at bias + 0x4B400000, which is
// 1.5 * 2^23 + sum as a float.  Three stacks at 16384 states, in turn on one card: 583, 592, 594 -> 576, 581, 585 us.  A
// bias can take a layer out of these ranges (no weights of these sizes can); such a network converts.
constexpr int ST_MAGIC = 0x4B400000;

// The workgroups of a unit take turns at being first.  Between wavefronts of equal priority a SIMD issues the oldest one's instructions, so
// the workgroup that came first runs through its images and leaves the unit to the others, which cannot fill it: of two (first stack, 16384
// states) one was through after 202 us and the other after 308, of four (second stack) after 99, 116, 157 and 179.  A turn is 2^LOG clocks
// of the unit's counter, which all see alike; the third stack, whose workgroups do not come in equal numbers, gains nothing.
// Traces in turn on one card, us, without / with: first stack 2048 states 49.7 / 48.1, 4096 95.2 / 92.6, 16384 335 / 326; second 31.6 / 30.4,
// 57.6 / 56.0, 194 / 181 (turns of 2^12 335 / 187 at 16384 states, 2^16 as long as 2^15).
template <int SLOTS, int LOG>
__device__ __forceinline__ void st_turn(int slot) {
    const int t = ((int)(__builtin_readcyclecounter() >> LOG) + slot) & (SLOTS - 1);
    if (t == 0) __builtin_amdgcn_s_setprio(0);
    else if (t == 1) __builtin_amdgcn_s_setprio(1);
    else if (t == 2) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(3);
}
template <bool BITS>
__device__ __forceinline__ float st_float(int acc) { return BITS ? __int_as_float(acc) - 12582912.0f : (float)acc; }

template <bool U8, int CI, int HIN, int C, int G, int SEG, int PSEG, int NW, int WL, int MINB, bool BITS>
__global__ __launch_bounds__(NW * 64, MINB) void stack_kernel(const StackParams p) {
    typedef StShape<U8, CI, HIN, C, G, SEG, PSEG, NW, WL> S;
    constexpr int T = S::THREADS;
    typedef int v2i __attribute__((ext_vector_type(2)));
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* tin = smem;                                    // G bordered input tiles
    char* tX = smem + S::O_TX;                           // G bordered tiles of max(stream, 0)
    char* tM = smem + S::O_TM;                           // G bordered tiles of the pooled stream, then of a block's inner tensor
    int* cst = (int*)(smem + S::O_CST);                  // [conv][bias 16 | mult 16]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;

    // ---- staging: unit u of the batch is one dword of each of the four planes, or 16 bytes of the images
    v4i pre[S::PF];
    int doff[S::PF];
#pragma unroll
    for (int i = 0; i < S::PF; ++i) {
        const int u = min(tid + i * T, G * S::UNITS_IN - 1);
        const int img = u / S::UNITS_IN, w = u - img * S::UNITS_IN, row = w / S::UPR_IN, cu = w - row * S::UPR_IN;
        doff[i] = img * S::TILE_IN + (row + 1) * S::PITCH_IN + CI + cu * 16;
    }
    const int64_t n_batch = (p.B + G - 1) / G;
    auto prefetch = [&](int64_t batch) {
        const int64_t b0 = batch * G;
        const int gc = (int)((p.B - b0 < G) ? (p.B - b0) : G);
        // (buffer loads: an observation's plane is their scalar offset; of int8 images, a unit that does not exist is out of the buffer's
        // range and reads 0)
        static_assert(!U8 || st_units_in_plane<S>(HIN * HIN), "no lane reads past a plane");
        const auto src = __builtin_amdgcn_make_buffer_rsrc((char*)p.in + (U8 && p.rows ? (int64_t)p.rows[b0] : b0) * (int64_t)S::IMG_IN, 0,
                                                           gc * S::IMG_IN, 0x00027000);
#pragma unroll
        for (int i = 0; i < S::PF; ++i) {
            if constexpr (U8) {
                v4i v;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = (int)__builtin_amdgcn_raw_buffer_load_b32(src, 4 * S::unit(tid, i), c * HIN * HIN, 0);
                pre[i] = v;
            } else {
                pre[i] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(src, 16 * (tid + i * T), 0, 0));
            }
        }
    };
    auto commit = [&](int64_t batch) {
        const int64_t b0 = batch * G;
        const int total = (G == 1 || p.B - b0 >= G ? G : (int)(p.B - b0)) * S::UNITS_IN;
#pragma unroll
        for (int i = 0; i < S::PF; ++i) {
            if (tid + i * T >= total) break;
            const v4i v = pre[i];
            if constexpr (U8) {
                // one dword (4 pixels) of each plane -> four channels-last pixels, stored as obs - 128
                const uint32_t P0 = (uint32_t)v[0], P1 = (uint32_t)v[1], P2 = (uint32_t)v[2], P3 = (uint32_t)v[3];
                const uint32_t lo01 = __builtin_amdgcn_perm(P1, P0, 0x05010400u), hi01 = __builtin_amdgcn_perm(P1, P0, 0x07030602u);
                const uint32_t lo23 = __builtin_amdgcn_perm(P3, P2, 0x05010400u), hi23 = __builtin_amdgcn_perm(P3, P2, 0x07030602u);
                uint32_t* d = (uint32_t*)(tin + doff[i]);
                d[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u) ^ 0x80808080u;
                d[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u) ^ 0x80808080u;
                d[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u) ^ 0x80808080u;
                d[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u) ^ 0x80808080u;
            } else if constexpr ((CI & 15) == 0) {
                *(v4i*)(tin + doff[i]) = v;
            } else {
                *(v2i*)(tin + doff[i]) = (v2i){v[0], v[1]};
                *(v2i*)(tin + doff[i] + 8) = (v2i){v[2], v[3]};
            }
        }
    };

    int64_t batch = blockIdx.x;
    // before the weights, so that a small call waits for both at once, and the borders meanwhile (third stack 8 states 9.6 -> 8.4 us, 1024 11.1 -> 10.1,
    // 4096 28.9 -> 26.6; first 160 states 11.8 -> 10.9)
    if (batch < n_batch) prefetch(batch);

    // ---- once per workgroup: borders (only interiors are written later), constants
    {
        const int padv = U8 ? (int)0x80808080u : 0;       // a padding pixel is the observation value 0
        for (int i = tid; i < S::O_TX / 16; i += T) ((v4i*)tin)[i] = (v4i){padv, padv, padv, padv};
        for (int i = tid; i < (S::O_W - S::O_TX) / 16; i += T) ((v4i*)tX)[i] = (v4i){0, 0, 0, 0};
        for (int i = tid; i < 5 * 16; i += T) {
            const int cv = i >> 4, n = i & 15;
            cst[cv * 32 + n] = p.bias[cv][n];
            ((float*)cst)[cv * 32 + 16 + n] = p.mult[cv][n];
        }
    }

    // ---- weights: those of the stack convolution and of the block convolutions WL .. 3 stay in registers, the others go to LDS
    v4i wP[S::NWP], wR[S::WL < 4 ? 4 - S::WL : 1][S::NWB];
    {
        // chunk (ky, cx) of the planner's fragments (cpr chunks per kernel row), zero outside the kernel
        auto chunk = [&](int cv, int cpr, int ky, int cx, int mrow) -> v4i {
            const bool in = ky >= 0 && ky < 3 && cx >= 0 && cx < cpr;
            const int q = in ? ky * cpr + cx : 0;
            const v4i v = p.w[cv][(q >> 2) * 64 + 16 * (q & 3) + mrow];
            return in ? v : (v4i){0, 0, 0, 0};
        };
        if constexpr (S::P == 2) {
            // a window is four input rows of four pixels, a row per lane group: the upper and the lower conv row under it.
            // MFMA rows 4 g .. 4 g + 3: the even column of channels 2 g, 2 g + 1, then the odd one (the planner's rows are
            // the eight channels of the even column, then of the odd one)
            const int jr = 8 * ((j >> 1) & 1) + 2 * (j >> 2) + (j & 1);
            wP[0] = chunk(0, S::CPR_C, g, 0, jr);
            wP[1] = chunk(0, S::CPR_C, g - 1, 0, jr);
        } else if constexpr (CI == 8) {
            // four input rows of four pixels in two steps of two rows: [E | O][upper | lower][step]
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int ky = 2 * (e & 1) + (g >> 1) - ((e >> 1) & 1), cx = g & 1;
                const v4i own = chunk(0, S::CPR_C, ky, cx, j), prev = chunk(0, S::CPR_C, ky, cx - 1, j);   // a chunk is two pixels
                wP[e] = e < 4 ? own : (v4i){prev[2], prev[3], own[0], own[1]};
            }
        } else {
            // an input row of four pixels per step: [E | O][ky]
#pragma unroll
            for (int e = 0; e < 6; ++e) wP[e] = chunk(0, S::CPR_C, e % 3, e < 3 ? g : g - 1, j);        // a pixel is a whole chunk
        }
        auto block = [&](v4i (&w)[S::NWB], int cv) {
            if constexpr (S::P == 2) {
                // four rows of four pixels in two steps of two rows serve two output rows: [upper | lower][step]
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = chunk(cv, S::CPR_B, 2 * (e & 1) + (g >> 1) - (e >> 1), g & 1, j);
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e) w[e] = chunk(cv, S::CPR_B, e, g, j);                        // a row of three pixels per step
            }
        };
#pragma unroll
        for (int cv = S::WL; cv < 4; ++cv) block(wR[cv - S::WL], cv + 1);
        for (int cv = wave; cv < S::WL; cv += NW) {
            v4i w[S::NWB];
            block(w, cv + 1);
#pragma unroll
            for (int e = 0; e < S::NWB; ++e)
                if (S::P == 2 || g < 3) *(v4i*)(smem + S::O_W + cv * S::WB + e * (S::WB / S::NWB) + lane * 16) = w[e];
        }
    }
    const int woff = S::O_W + (S::P == 2 ? lane : 16 * min(g, 2) + j) * 16;
    auto weights = [&](auto conv, v4i (&w)[S::NWB]) {    // fragments of block convolution 0 .. 3
        constexpr int cv = decltype(conv)::value;
#pragma unroll
        for (int e = 0; e < S::NWB; ++e)
            if constexpr (cv >= S::WL) w[e] = wR[cv - S::WL][e];
            else w[e] = *(const v4i*)(smem + woff + cv * S::WB + e * (S::WB / S::NWB));
    };
    // the weights are in their registers before the loop: the waits the compiler places there then only ever concern the
    // loads of the next batch, not these
    __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)

    // ---- this lane's column of the blocks; lanes past the last column repeat it (the same bytes written twice)
    const int n = wave * 16 + j, nc = min(n, S::NCOL - 1);
    const int bimg = nc / (SEG * S::WP), bseg = (nc - bimg * SEG * S::WP) / S::WP, bcol = nc - (bimg * SEG + bseg) * S::WP;
    const int row0 = bseg * S::R;
    const int bpos = bimg * S::TILE_B + row0 * S::PITCH_B + bcol * 16;
    // (16-channel layers have no fourth chunk: its lanes read the zeros of the left border)
    const int boff = S::P == 2 ? bpos + (g >> 1) * S::PITCH_B + (g & 1) * 16 : g < 3 ? bpos + g * 16 : bpos - bcol * 16;
    const int bown = bpos + S::PITCH_B + C + 4 * g;       // the column's own pixel(s) sit one row and one pixel inside its window
    const int brel = (row0 * S::WP + bcol) * 16 + 4 * g;  // in a plain image
    // ---- this lane's column of the pooling (16-channel layers): slots are the column runs (image, segment), each behind a
    //      dummy that repeats its first pixel; a tile's first lane repeats the last slot of the tile before it
    int ppos = 0, pout = 0, pfirst = 0;
    if constexpr (S::P == 1) {
        const int s = min(15 * wave + j, S::SLOTS - 1) + 1, run = s / (S::H + 1), at = s - run * (S::H + 1);
        const int px = max(at - 1, 0), img = run / PSEG, p0 = min((run - img * PSEG) * S::RP, S::H - S::RP);
        const bool st = at > 0 && 15 * wave + j < S::SLOTS && (wave == 0 || j > 0);
        // (odd sizes: the last pooled pixel's columns are the last two, its window starts a pixel earlier)
        const int wx = 2 * px - ((HIN & 1) && px == S::H - 1 ? 1 : 0);
        ppos = img * S::TILE_IN + 2 * p0 * S::PITCH_IN + wx * CI + (CI == 8 ? (g >> 1) * S::PITCH_IN + (g & 1) * 16 : g * 16);
        pfirst = p0 > 0 ? -2 * S::PITCH_IN : 0;            // the window above, for the conv row shared with it
        pout = img * S::TILE_B + (p0 + 1) * S::PITCH_B + (st ? px + 1 : S::H + 2) * C + 4 * g;
    }
    __syncthreads();

    const int slot = blockIdx.x / (uint32_t)p.units;
    auto turn = [&]() {
        if constexpr (S::P == 2) st_turn<2, 14>(slot);
        else if constexpr (CI == 8) st_turn<4, 13>(slot);
    };
    for (; batch < n_batch; batch += gridDim.x) {
        turn();
        commit(batch);
        __syncthreads();
        const int64_t b0 = batch * G;
        const int gc = (int)((p.B - b0 < G) ? (p.B - b0) : G);

        // ---- stack convolution + max-pool, in registers -> bordered tiles of max(x, 0) and of x itself
        {
            v4i biC = *(const v4i*)(cst + 4 * g) + (BITS ? ST_MAGIC : 0);
            v4f mlC = *(const v4f*)(cst + 16 + 4 * g);
            if constexpr (S::P == 2) {                   // channels 2 g, 2 g + 1 twice
                const int b0 = cst[2 * g] + (BITS ? ST_MAGIC : 0), b1 = cst[2 * g + 1] + (BITS ? ST_MAGIC : 0);
                const float m0 = ((const float*)cst)[16 + 2 * g], m1 = ((const float*)cst)[16 + 2 * g + 1];
                biC = (v4i){b0, b1, b0, b1};
                mlC = (v4f){m0, m1, m0, m1};
            }
            auto requant = [&](const int (&pooled)[4]) {
                int q[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) q[r] = rne_clamp127(st_float<BITS>(pooled[r]) * mlC[r]);
                return st_pack(q);
            };
            if constexpr (S::P == 2) {
                // work item: (pair of pooled rows, strip of 15 pixels behind the one that only serves its neighbour).  A wavefront
                // walks down runs of them: an item's windows are two fragments, and the lower conv row of the row above is the
                // last product of the item before.  Runs that cross into the next strip do so at few places of the unrolled walk.
                constexpr int NS = (S::H - 1 + 14) / 15, RPS = S::H / 2, N_IT = RPS * NS, PER = (N_IT + NW - 1) / NW;
                static_assert(N_IT >= NW * PER - 1 && PER <= RPS, "runs: only the last one may be short, by its last item");
                constexpr auto crosses = [](int i) {
                    for (int w = 0; w < NW; ++w) if (i > 0 && (w * PER + i) % RPS == 0) return true;
                    return false;
                };
                const int it0 = wave * PER;
                int s = it0 / RPS, left = RPS - (it0 - s * RPS);      // (the strip, its items that are left)
                const char* a;
                char* o;
                auto strip = [&](int rp) {                            // at row pair rp of strip s
                    a = tin + j * 2 * CI + g * S::PITCH_IN + s * 30 * CI + 4 * rp * S::PITCH_IN;
                    const bool ok = (s == 0 || j > 0) && (s < NS - 1 || 15 * (NS - 1) + j < S::H);
                    o = tX + 2 * g + (2 * rp + 1) * S::PITCH_B + (ok ? (s * 15 + 1 + j) * C : (S::H + 2) * C);
                };
                strip(RPS - left);
                v4i c0 = st_mfma(wP[1], read_chunk<8>(a - (left < RPS ? 2 * S::PITCH_IN : 0)), biC);
                int at = 0;                                           // the item that a and o belong to
                auto window = [&](int i) { return read_chunk<8>(a + i * 2 * S::PITCH_IN); };
                v4i f0 = window(0), f1 = window(1);
#pragma unroll
                for (int i = 0; i < PER; ++i) {
                    if (crosses(i)) {
                        if (left == i) {                              // the first row's window has no row above it: its own upper one again
                            ++s;
                            strip(0);
                            f0 = window(0);
                            f1 = window(1);
                            c0 = st_mfma(wP[1], f0, biC);
                        } else {
                            a += 4 * (i - at) * S::PITCH_IN;
                            o += 2 * (i - at) * S::PITCH_B;
                        }
                        at = i;
                    }
                    if (N_IT % PER && i == PER - 1 && it0 + i >= N_IT) break;
                    const v4i c1 = st_mfma(wP[0], f0, biC), c2 = st_mfma(wP[1], f0, biC), c3 = st_mfma(wP[0], f1, biC), c4 = st_mfma(wP[1], f1, biC);
                    // the next item's, before this one's results are stored (past the strip's end: something, and not used)
                    if (i + 1 < PER) { f0 = window(2 * (i + 1 - at)); f1 = window(2 * (i + 1 - at) + 1); }
                    // a lane holds two channels of both columns: upper pooled row in pooled[0], [1], lower in [2], [3]
                    int vo[4] = {max(max(c0[2], c1[2]), c2[2]), max(max(c0[3], c1[3]), c2[3]), max(max(c2[2], c3[2]), c4[2]), max(max(c2[3], c3[3]), c4[3])};
                    max_with_left(vo);
                    const int pooled[4] = {max(max(max(c0[0], c1[0]), c2[0]), vo[0]), max(max(max(c0[1], c1[1]), c2[1]), vo[1]),
                                           max(max(max(c2[0], c3[0]), c4[0]), vo[2]), max(max(max(c2[1], c3[1]), c4[1]), vo[3])};
                    c0 = c4;
                    const StBytes w = requant(pooled);
                    char* d = o + 2 * (i - at) * S::PITCH_B;
                    *(uint16_t*)d = (uint16_t)w.pos;
                    *(uint16_t*)(d + S::PITCH_B) = (uint16_t)(w.pos >> 16);
                    *(uint16_t*)(d + S::O_TM - S::O_TX) = (uint16_t)w.raw;
                    *(uint16_t*)(d + S::O_TM - S::O_TX + S::PITCH_B) = (uint16_t)(w.raw >> 16);
                }
            } else if (wave < S::NT1) {
                auto out = [&](int k, v4i e, v4i o) {
                    int vo[4] = {o[0], o[1], o[2], o[3]}, pooled[4];
                    max_with_left(vo);
#pragma unroll
                    for (int r = 0; r < 4; ++r) pooled[r] = max(e[r], vo[r]);
                    const StBytes w = requant(pooled);
                    *(uint32_t*)(tX + pout + k * S::PITCH_B) = w.pos;
                    *(uint32_t*)(tM + pout + k * S::PITCH_B) = w.raw;
                };
                auto max3 = [](v4i x, v4i y, v4i z) {
                    v4i m;
#pragma unroll
                    for (int r = 0; r < 4; ++r) m[r] = max(max(x[r], y[r]), z[r]);
                    return m;
                };
                const char* a = tin + ppos;
                if constexpr (CI == 8) {
                    auto conv = [&](const v4i* w, v4i lo, v4i hi) { return st_mfma(w[1], hi, st_mfma(w[0], lo, biC)); };
                    v4i f0 = *(const v4i*)a;
                    // the lower conv row of the window above (for the first pooled row: of its own window)
                    v4i cE, cO;
                    {
                        const v4i m0 = *(const v4i*)(a + pfirst), m1 = *(const v4i*)(a + pfirst + 2 * S::PITCH_IN);
                        cE = conv(wP + 2, m0, m1);
                        cO = conv(wP + 6, m0, m1);
                    }
#pragma unroll
                    for (int k = 0; k < S::RP; ++k) {
                        const v4i f1 = *(const v4i*)(a + (2 * k + 2) * S::PITCH_IN);
                        const v4i e0 = conv(wP, f0, f1), e1 = conv(wP + 2, f0, f1), o0 = conv(wP + 4, f0, f1), o1 = conv(wP + 6, f0, f1);
                        out(k, max3(cE, e0, e1), max3(cO, o0, o1));
                        cE = e1; cO = o1; f0 = f1;
                    }
                } else {
                    static_assert(S::AHEAD, "16 input channels");
                    auto conv = [&](const v4i* w, v4i r0, v4i r1, v4i r2) { return st_mfma(w[2], r2, st_mfma(w[1], r1, st_mfma(w[0], r0, biC))); };
                    auto row = [&](int y) { return *(const v4i*)(a + y * S::PITCH_IN); };
                    constexpr auto below = [](int k) { return !(HIN & 1) || k + 1 < S::RP; };    // (odd sizes: no conv row below the last)
                    v4i f0 = row(0), f1 = row(1), f2 = row(2), f3 = row(3), cE, cO;
                    {
                        const char* m = a + pfirst;
                        const v4i m1 = *(const v4i*)(m + S::PITCH_IN), m2 = *(const v4i*)(m + 2 * S::PITCH_IN), m3 = *(const v4i*)(m + 3 * S::PITCH_IN);
                        cE = conv(wP, m1, m2, m3);
                        cO = conv(wP + 3, m1, m2, m3);
                    }
                    v4i e0 = conv(wP, f0, f1, f2), o0 = conv(wP + 3, f0, f1, f2), e1 = conv(wP, f1, f2, f3), o1 = conv(wP + 3, f1, f2, f3);
                    f0 = f2; f1 = f3; f2 = row(4); f3 = row(5);
#pragma unroll
                    for (int k = 0; k < S::RP; ++k) {
                        const v4i mE = max3(cE, e0, e1), mO = max3(cO, o0, o1);
                        cE = e1; cO = o1;
                        if (k + 1 < S::RP) {
                            e0 = conv(wP, f0, f1, f2); o0 = conv(wP + 3, f0, f1, f2);
                            e1 = e0; o1 = o0;
                            if (below(k + 1)) { e1 = conv(wP, f1, f2, f3); o1 = conv(wP + 3, f1, f2, f3); }
                            f0 = f2; f1 = f3;
                            if (k + 2 < S::RP) { f2 = row(2 * k + 6); if (below(k + 2)) f3 = row(2 * k + 7); }
                        }
                        out(k, mE, mO);
                        if (k + 1 < S::RP) {
#pragma unroll
                            for (int m = 0; m < (below(k + 1) ? 12 : 6); ++m) {
                                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
        __syncthreads();

        // ---- one block convolution: walk down this lane's column; done(k, acc) takes output row k in V vector instructions
        auto walk = [&](const char* src, const v4i (&w)[S::NWB], v4i b, auto per_row, auto&& done) {
            constexpr int V = decltype(per_row)::value;
            const char* a = src + boff;
            auto row = [&](int y) { return *(const v4i*)(a + y * S::PITCH_B); };
            if constexpr (S::P == 2) {
                v4i f0 = row(0);
#pragma unroll
                for (int k = 0; k < S::R; k += 2) {
                    const v4i f1 = row(k + 2);
                    const v4i u = st_mfma(w[1], f1, st_mfma(w[0], f0, b));
                    if (k + 1 < S::R) {
                        const v4i l = st_mfma(w[3], f1, st_mfma(w[2], f0, b));
                        done(k, u);
                        done(k + 1, l);
                    } else {
                        done(k, u);
                    }
                    f0 = f1;
                }
            } else if constexpr (!S::AHEAD) {
                v4i f0 = row(0), f1 = row(1);
#pragma unroll
                for (int k = 0; k < S::R; ++k) {
                    const v4i f2 = row(k + 2);
                    done(k, st_mfma(w[2], f2, st_mfma(w[1], f1, st_mfma(w[0], f0, b))));
                    f0 = f1; f1 = f2;
                }
            } else {
                v4i f0 = row(0), f1 = row(1), f2 = row(2), f3 = row(3);
                v4i acc = st_mfma(w[2], f2, st_mfma(w[1], f1, st_mfma(w[0], f0, b)));
#pragma unroll
                for (int k = 0; k < S::R; ++k) {
                    v4i next = acc, f4 = f3;
                    if (k + 1 < S::R) {
                        if (k + 2 < S::R) f4 = row(k + 4);
                        next = st_mfma(w[2], f3, st_mfma(w[1], f2, st_mfma(w[0], f1, b)));
                    }
                    done(k, acc);
                    if (k + 1 < S::R) {
#pragma unroll
                        for (int m = 0; m < 3; ++m) {
                            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                            if (m == 0 && k + 2 < S::R) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                            __builtin_amdgcn_sched_group_barrier(0x002, V / 3, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    acc = next; f1 = f2; f2 = f3; f3 = f4;
                }
            }
        };
        // ---- a block's first convolution: max(x, 0) -> inner tensor, requantized with the fused ReLU
        auto conv_a = [&](const v4i (&w)[S::NWB], int cv) {
            const v4i bi = *(const v4i*)(cst + cv * 32 + 4 * g) + (BITS ? P23_MAGIC : 0);
            const v4f ml = *(const v4f*)(cst + cv * 32 + 16 + 4 * g);
            const v4f cc = ml * -8388608.0f;
            walk(tX, w, bi, std::integral_constant<int, BITS ? 12 : 16>{}, [&](int k, v4i acc) {
                const uint32_t y = requant_relu4_p23<BITS>(acc, ml, cc);
                *(uint32_t*)(tM + bown + k * S::PITCH_B) = y;
            });
        };
        uint32_t x[S::R];                                 // the stream under this lane, four channels per row
        // ---- a block's second convolution, joined with the block's input; LAST: to memory, else back into registers and LDS
        auto conv_b = [&](const v4i (&w)[S::NWB], int cv, float rr, auto last) {
            constexpr bool LAST = decltype(last)::value;
            const v4i bi = *(const v4i*)(cst + cv * 32 + 4 * g) + (BITS ? ST_MAGIC : 0);
            const v4f ml = *(const v4f*)(cst + cv * 32 + 16 + 4 * g);
            asm("" : "+v"(rr));                           // a vector register: a multiplication by a scalar one takes twice as long
            char* outp = (char*)p.out + b0 * (int64_t)S::IMG + (uint32_t)(bimg * S::IMG + brel);
            // (a short last batch: the buffer ends with its last image, and what lanes of missing ones store behind it is dropped.  A
            // branch around the phase would leave the matrix instructions with some of a wavefront's lanes only.  Rows by the scalar
            // offset: added to the lanes' they took a register and an instruction each)
            const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((char*)p.out + b0 * (int64_t)S::IMG, 0, gc * S::IMG, 0x00027000);
            walk(tM, w, bi, std::integral_constant<int, LAST ? 27 : 29>{}, [&](int k, v4i acc) {
                int q[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float tr = (float)(int)(int8_t)(x[k] >> (8 * r)) * rr;
                    q[r] = rne_clamp127(fmaf(st_float<BITS>(acc[r]), ml[r], tr));
                }
                const StBytes y = st_pack(q);
                if constexpr (LAST) {
                    if constexpr (G > 1) __builtin_amdgcn_raw_buffer_store_b32(y.raw, rsrc, bimg * S::IMG + brel, k * S::WP * 16, 0);
                    else *(uint32_t*)(outp + k * S::WP * 16) = y.raw;
                } else {
                    x[k] = y.raw;
                    *(uint32_t*)(tX + bown + k * S::PITCH_B) = y.pos;
                }
            });
        };
        // The pooled stream waits where the inner tensor will be: its pixels' owners take it into registers before they
        // write there, and it stays in registers from then on.
        turn();
        v4i wA[S::NWB], wB[S::NWB];
#pragma unroll
        for (int k = 0; k < S::R; ++k) x[k] = *(const uint32_t*)(tM + bown + k * S::PITCH_B);
        weights(std::integral_constant<int, 0>{}, wA);
        conv_a(wA, 1);
        weights(std::integral_constant<int, 1>{}, wB);
        __syncthreads();
        conv_b(wB, 2, p.r1, std::false_type{});
        weights(std::integral_constant<int, 2>{}, wA);
        turn();
        __syncthreads();
        conv_a(wA, 3);
        weights(std::integral_constant<int, 3>{}, wB);
        __syncthreads();
        // the next batch's bytes are requested here, not earlier: their registers are then free during the phases above
        // (where the kernel needs the most), and the last phase is long enough for the loads to land
        if (batch + gridDim.x < n_batch) prefetch(batch + gridDim.x);
        if (G == 1 || __builtin_amdgcn_ballot_w64(bimg < gc)) conv_b(wB, 4, p.r2, std::true_type{});
        // no barrier here: the next commit writes the input tiles only, and the barrier behind it comes before the
        // next batch writes anything that the last phase reads
    }
}

// the five convolutions of a stack as the planner laid them out: c = stack convolution (with its fused pool),
// a1 / b1 and a2 / b2 = the two blocks
template <bool U8, int CI, int HIN, int C, int G, int SEG, int PSEG, int NW, int WL>
bool st_shape_ok(const ConvParams& c, const ConvParams& a1, const ConvParams& b1, const ConvParams& a2, const ConvParams& b2) {
    typedef StShape<U8, CI, HIN, C, G, SEG, PSEG, NW, WL> S;
    if (c.H != HIN || c.W != HIN || c.Cs_in != CI || c.Cin_real != CI || c.Ho != HIN || c.Wo != HIN / S::P || c.Cs_out != 16) return false;
    if (c.k != 3 || c.s != 1 || c.pad != 1 || c.sx != S::P || c.cpr != S::CPR_C || c.k_steps != S::KS_C) return false;
    if ((c.src_u8 != 0) != U8 || !c.pool || c.PH != S::H || c.PW != S::H || c.relu || c.relu_in || c.out_frag) return false;
    for (const ConvParams* b : {&a1, &b1, &a2, &b2}) {
        if (b->H != S::H || b->W != S::H || b->Cin_real != C || b->Cs_in != C || b->Ho != S::H || b->Wo != S::WP || b->Cs_out != 16) return false;
        if (b->k != 3 || b->s != 1 || b->pad != 1 || b->sx != S::P || b->cpr != S::CPR_B || b->k_steps != S::KS_B) return false;
        if (b->src_u8 || b->pool || b->out_frag) return false;
    }
    return a1.relu_in && a1.relu && !b1.relu_in && !b1.relu && a2.relu_in && a2.relu && !b2.relu_in && !b2.relu;
}

template <bool U8, int CI, int HIN, int C, int G, int SEG, int PSEG, int NW, int WL, int MINB, bool BITS>
hipError_t st_go(const StackParams& p, hipStream_t s) {
    typedef StShape<U8, CI, HIN, C, G, SEG, PSEG, NW, WL> S;
    auto kfn = stack_kernel<U8, CI, HIN, C, G, SEG, PSEG, NW, WL, MINB, BITS>;
    static int occ = 0;
    if (!occ) {
        hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS);
        if (e != hipSuccess) return e;
        int o = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, (const void*)kfn, S::THREADS, S::LDS);
        if (e != hipSuccess) return e;
        occ = o < 1 ? 1 : o;
    }
    // resident workgroups striding over the batches, in even rounds
    const int64_t batches = (p.B + G - 1) / G;
    const int64_t cap = (int64_t)occ * conv_num_cus();
    const int64_t rounds = (batches + cap - 1) / cap;
    dim3 grid((unsigned)((batches + rounds - 1) / rounds));
    kfn<<<grid, dim3(S::THREADS), S::LDS, s>>>(p);
    return hipGetLastError();
}

}  // namespace

// (uint8 source, stored input channels, input size, channels, images per batch, row segments of the blocks' and of the pool's
// lanes, wavefronts per workgroup, block convolutions whose weights live in LDS, wavefronts per SIMD the register budget is
// set for).  Measured at 16384 states: the second stack as two images in eight wavefronts 212 us (its barriers hold twice as
// many), with 16 wavefronts per unit instead of 12 182 for 196; the third with five images in four wavefronts 72 us (55 of 64
// lanes and 59 of 61 pooling slots in use), four images 79, four in eight wavefronts of two segments 88, two 94.
#define ACCERL_STACK_SHAPES(X) X(true, 4, 84, 8, 1, 6, 1, 8, 4, 4) X(false, 8, 42, 16, 1, 3, 2, 4, 3, 4) X(false, 16, 21, 16, 5, 1, 1, 4, 4, 2)

bool stack_supported(const ConvParams& c, int NTC, const ConvParams& a1, const ConvParams& b1, const ConvParams& a2, const ConvParams& b2) {
    if (NTC != 1) return false;
#define X(U8, CI, HIN, C, G, SEG, PSEG, NW, WL, MINB) if (st_shape_ok<U8, CI, HIN, C, G, SEG, PSEG, NW, WL>(c, a1, b1, a2, b2)) return true;
    ACCERL_STACK_SHAPES(X)
#undef X
    return false;
}

hipError_t launch_stack(const ConvParams& c, const ConvParams& a1, const ConvParams& b1, const ConvParams& a2, const ConvParams& b2, hipStream_t s) {
    if (c.B <= 0) return hipSuccess;
    StackParams p;
    p.in = c.in; p.rows = c.rows; p.out = (int8_t*)b2.out;
    const ConvParams* cv[5] = {&c, &a1, &b1, &a2, &b2};
    for (int i = 0; i < 5; ++i) { p.w[i] = (const v4i*)cv[i]->wfrag; p.bias[i] = (const int*)cv[i]->bias; p.mult[i] = cv[i]->mult; }
    p.r1 = b1.r; p.r2 = b2.r; p.B = c.B; p.units = (int)conv_num_cus();
    static const bool no_p23 = getenv("ACCERL_NO_P23") != nullptr;
    const bool bits = a1.pos23 && a2.pos23 && c.mag22 && b1.mag22 && b2.mag22 && !no_p23;
#define X(U8, CI, HIN, C, G, SEG, PSEG, NW, WL, MINB)                                                              \
    if (st_shape_ok<U8, CI, HIN, C, G, SEG, PSEG, NW, WL>(c, a1, b1, a2, b2))                                      \
        return bits ? st_go<U8, CI, HIN, C, G, SEG, PSEG, NW, WL, MINB, true>(p, s) : st_go<U8, CI, HIN, C, G, SEG, PSEG, NW, WL, MINB, false>(p, s);
    ACCERL_STACK_SHAPES(X)
#undef X
    return hipErrorInvalidValue;
}

}  // namespace accerl
