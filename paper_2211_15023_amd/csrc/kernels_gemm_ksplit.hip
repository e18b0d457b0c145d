// Dense layers whose wavefronts split K: a workgroup owns 16 * RT states x 16 * NT features, each of its eight wavefronts
// multiplies the whole tile over its own eighth of the MFMA steps with operands straight from memory, and the partial sums
// meet in LDS, where every wavefront finishes its share of the tiles.  The split of K and the order of the partial sums do
// not depend on the tile, so a state's result does not depend on the batch it is in.
//
// What bounds it: the fetches.  A compute unit pulls 25 to 45 bytes per clock out of the second-level cache and the memory behind it
// however many loads its wavefronts keep open, so the tile is the smallest that still gives every unit one workgroup: more units
// pull, and none of them twice; beyond that the largest, whose operands are fetched least often.  The kernel this replaces walked K alone in each 64 x 64 workgroup
// (64 workgroups on 256 units for 1024 states of a 3872 -> 256 layer): 41 -> 10.2 us there; 3136 -> 512 at 500 states
// 28 -> 8 us, at 4096 states 33 -> 28 us, 25 with two 64 x 64 tiles per unit, 18.7 with one of 128 x 64 (13 of it the fetches, 3 the partial
// sums in LDS).
#include <type_traits>

#include "gemm_epilogue.h"

namespace accerl {

int conv_num_cus();   // compute units of the current device

namespace {

constexpr int KS_LDS = 64 * 1024;
constexpr int KS_W = KSPLIT_PARTS;                            // wavefronts per workgroup

// The state's half of an LSTM operand (GemmParams::xh): thread tid of T packs 8-value pieces of ROWS states, those of the
// workgroup's share (y of ny) of h; as lstm_pack_frag_kernel.  The first piece is requested when the kernel starts and
// stored when it ends (one piece a thread is all there is for 64 x 64 tiles and as many units as inputs).  4096 states, 1936 -> 256
// in front of 256 units: 10.7 us and 5.2 for the packing kernel -> 12.2; bf16 3872 -> 256 at 999 states 10.5 + 3.8 -> 11.2.  Kernels of
// their own: carried by the plain ones as a test of p.xh, this cost every dense layer about a microsecond.
template <bool XH, int T, int ROWS>
struct LstmState {
    const GemmParams& p;
    int64_t b0, b;
    int tid, q0, np, items, q;
    v4f h0, h1;
    bool dn;
    __device__ __forceinline__ LstmState(const GemmParams& p_, int64_t b0_, unsigned y, int tid_) : p(p_), b0(b0_), tid(tid_), items(0) {
        if (!XH) return;
        const int Q = p.Hd >> 3;
        q0 = y * Q / gridDim.y;
        np = (y + 1) * Q / gridDim.y - q0;
        items = ROWS * np;
        if (tid < items) load(tid);
    }
    __device__ __forceinline__ void load(int i) {
        const int t = i >> 4, u = t / np;
        b = b0 + 16 * u + (i & 15);
        q = q0 + t - u * np;
        if (b >= p.B) return;
        const v4f* h = (const v4f*)(p.h + b * p.Hd + 8 * q);
        h0 = h[0]; h1 = h[1];
        dn = p.done && p.done[b] != 0;
    }
    __device__ __forceinline__ void store() {
        if (!XH) return;
        for (int i = tid; i < items; i += T) {
            if (i != tid) load(i);
            if (b >= p.B) continue;                        // (the product does not store these states)
            if (dn) {
                const v4f z = {0.0f, 0.0f, 0.0f, 0.0f};
                v4f *h = (v4f*)(p.h + b * p.Hd + 8 * q), *c = (v4f*)(p.c + b * p.Hd + 8 * q);
                h[0] = h0 = z; h[1] = h1 = z;
                c[0] = z; c[1] = z;
            }
            const float lo[4] = {h0[0], h0[1], h0[2], h0[3]}, hi[4] = {h1[0], h1[1], h1[2], h1[3]};
            const v2i l = lstm_pack4(lo), u = lstm_pack4(hi);
            *(v4i*)lstm_piece(p, b, p.N + 8 * q) = (v4i){l[0], l[1], u[0], u[1]};
        }
    }
};

template <int EL, int EPI, int RT, int NT, bool RELU, bool FRAG, bool XH>
__global__ __launch_bounds__(64 * KS_W) void gemm_ksplit_kernel(const GemmParams p) {
    typedef typename std::conditional<EL == EL_I8, v4i, v4f>::type Acc;
    constexpr int W = KS_W, D = 2;                          // D steps in flight per wavefront
    constexpr int FIT = KS_LDS / (W * NT * 1024);
    constexpr int RH = RT < FIT ? RT : FIT;                   // state tiles folded at a time
    __shared__ __attribute__((aligned(16))) Acc s_part[W * RH * NT * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const GemmTile tile = gemm_tile<!XH>(p.by_xcd);
    const int64_t b0 = (int64_t)tile.x * (16 * RT);
    const int nt0 = tile.y * NT;
    const int ks = p.k_steps;
    const int s0 = wave * ks / W, s1 = (wave + 1) * ks / W;   // this wavefront's steps
    LstmState<XH, 64 * W, 16 * RT> lstm(p, b0, tile.y, tid);

    // Row-major states: a lane fetches 16 bytes of row lane / 4 (four lanes read 64 consecutive bytes; the fragment's own order
    // would touch 16 rows per quarter wavefront), and the wavefront turns them into fragments through its own LDS region.
    // States past the batch re-read the last one (or the last tile), features past the last tile re-read the first one;
    // neither is stored.
    const int xc = lane & 3;                                   // which 16 bytes of a step this lane fetches
    v4i* turn = (v4i*)s_part + wave * RT * 64;
    const int turn_w = (lane >> 2) * 4 + (xc ^ (lane >> 4)), turn_r = j * 4 + (g ^ (j >> 2));   // no bank conflicts either way
    const char* xb = (const char*)p.x + (FRAG ? (b0 >> 4) * ((int64_t)ks << 10) : b0 * p.Kp_bytes);
    const int left = (int)min(p.B - b0, (int64_t)(16 * RT));
    uint32_t xo[RT];
#pragma unroll
    for (int u = 0; u < RT; ++u)
        xo[u] = FRAG ? (uint32_t)min(u, (left - 1) >> 4) * ((uint32_t)ks << 10) + lane * 16
                     : (uint32_t)min(16 * u + (lane >> 2), left - 1) * (uint32_t)p.Kp_bytes;
    const char* wb = (const char*)p.wfrag + (int64_t)nt0 * ks * 1024;
    uint32_t wo[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) wo[t] = (uint32_t)(nt0 + t < p.n_tiles ? t : 0) * ((uint32_t)ks << 10) + lane * 16;

    Acc acc[RT][NT];
#pragma unroll
    for (int u = 0; u < RT; ++u)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[u][t] = (Acc){0, 0, 0, 0};
    auto load = [&](int step, v4i (&a)[NT], v4i (&x)[RT]) {
        const uint32_t st = (uint32_t)min(step, ks - 1);      // past the end: a valid step, not multiplied
        uint32_t kb = st * 1024;
        if (!FRAG) kb = min(st * 64 + 16 * xc, ((uint32_t)p.Kp_bytes - 16) & ~3u);
#pragma unroll
        for (int t = 0; t < NT; ++t) a[t] = *(const v4i*)(wb + (wo[t] + (st << 10)));
#pragma unroll
        for (int u = 0; u < RT; ++u) x[u] = *(const v4i*)(xb + (xo[u] + kb));
    };
    auto mul = [&](int step, const v4i (&a)[NT], v4i (&x)[RT]) {
        if (!FRAG && (step + 1) * 64 > p.Kp_bytes) {
            // the end of the rows: a chunk past it becomes zeros (its weights are), one that straddles it re-read the row's
            // last 16 bytes and is rebuilt from those that belong to it
            const int have = p.Kp_bytes - (step * 64 + 16 * xc);
            const int sh = have >= 16 ? 0 : have > 0 ? (16 - have) >> 2 : 4;
#pragma unroll
            for (int u = 0; u < RT; ++u) {
                const v4i v = x[u];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    int r = 0;
#pragma unroll
                    for (int k = e; k < 4; ++k) r = k - e == sh ? v[k] : r;
                    x[u][e] = r;
                }
            }
        }
        if (RELU) {
#pragma unroll
            for (int u = 0; u < RT; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) x[u][e] = (int)(EL == EL_I8 ? g_relu_i8x4((uint32_t)x[u][e]) : g_relu_bf16x2((uint32_t)x[u][e]));
        }
        if (!FRAG) {
#pragma unroll
            for (int u = 0; u < RT; ++u) turn[u * 64 + turn_w] = x[u];
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // lanes read what other lanes of the wavefront wrote
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int u = 0; u < RT; ++u) x[u] = turn[u * 64 + turn_r];
            __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (EL == EL_I8) acc[u][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t], x[u], acc[u][t], 0, 0, 0);
                else acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a[t]), __builtin_bit_cast(v8bf, x[u]), acc[u][t], 0, 0, 0);
            }
    };
    if constexpr (RT == 8 && FRAG) {
        // One step in flight: a state fragment is requested again as soon as its products are issued, the weights a step ahead.  Two whole
        // steps a wavefront (192 KB a unit) fetch 31 bytes a clock and unit where one fetches 43 (the loads alone, 3136 -> 512 at 4096 states).
        v4i a[2][NT], x[RT];
        auto load_a = [&](int step, v4i (&v)[NT]) {
            const uint32_t st = (uint32_t)min(step, ks - 1) << 10;
#pragma unroll
            for (int t = 0; t < NT; ++t) v[t] = *(const v4i*)(wb + (wo[t] + st));
        };
        auto load_x = [&](int step, int u) { x[u] = *(const v4i*)(xb + (xo[u] + ((uint32_t)min(step, ks - 1) << 10))); };
        load_a(s0, a[0]);
#pragma unroll
        for (int u = 0; u < RT; ++u) load_x(s0, u);
        for (int st = s0; st < s1; st += 2) {
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                load_a(st + d + 1, a[d ^ 1]);
                if (d && st + d >= s1) break;
#pragma unroll
                for (int u = 0; u < RT; ++u) {
                    if (RELU) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[u][e] = (int)g_relu_bf16x2((uint32_t)x[u][e]);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t)
                        acc[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a[d][t]), __builtin_bit_cast(v8bf, x[u]), acc[u][t], 0, 0, 0);
                    load_x(st + d + 1, u);
                    __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
            }
        }
    } else {
        v4i a[D][NT], x[D][RT];
#pragma unroll
        for (int d = 0; d < D; ++d) load(s0 + d, a[d], x[d]);
        for (int st = s0; st < s1; st += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (st + d < s1) mul(st + d, a[d], x[d]);
                load(st + D + d, a[d], x[d]);
            }
        }
    }

#pragma unroll
    for (int u0 = 0; u0 < RT; u0 += RH) {
        if (!FRAG || u0) __syncthreads();                      // the regions above are free, the tiles before have been folded
#pragma unroll
        for (int u = 0; u < RH; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) s_part[((wave * RH + u) * NT + t) * 64 + lane] = acc[u0 + u][t];
        __syncthreads();
        for (int i = wave; i < RH * NT; i += W) {
            const int u = i / NT, t = i - u * NT;
            const int64_t b = b0 + 16 * (u0 + u) + j;
            const int n0 = (nt0 + t) * 16 + 4 * g;
            if (nt0 + t >= p.n_tiles || b >= p.B || n0 >= p.Np) continue;
            Acc sum = *(const Acc*)((const char*)p.bias + 4 * n0);
#pragma unroll
            for (int w = 0; w < W; ++w) sum += s_part[((w * RH + u) * NT + t) * 64 + lane];
            gemm_finish<EPI, XH>(p, sum, b, n0);
        }
    }
    lstm.store();
}

// An eighth more than one workgroup per compute unit: where the three rules below that name it end (pick's tiles end at one).
int64_t most_groups() { return conv_num_cus() * 9 / 8; }

// Whether gemm_tile orders by XCD.  In the grid's own order the workgroups of one group of states meet on an XCD only if the groups are a
// multiple of eight; else each is fetched by up to eight (whole forwards, us, grid / XCD: 3136 -> 512 bf16 200 states 25.8 / 23.9, 400
// 31.3 / 28.8, 3600 110 / 97, int8 400 22.5 / 20.7, 900 29.5 / 27.4; 3600 -> 500 bf16 3900 83.2 / 60.6).  With a multiple of eight, or one
// workgroup over all features, nothing is gained in the product, and the convolution in front of it takes longer (2304 -> 256 bf16 at 4096
// states 20.2 / 22.9, whole forwards 35.0 / 37.0, at 2048 24.6 / 25.9; -> 24 at 3000, 188 groups, 23.7 / 26.3) -- except beyond one round,
// where a group's first and last features no longer run together, as long as the weights then stay in the 4 MB of an XCD's second-level
// cache (3600 -> 500 at 16384 states 186 / 173, 2304 -> 512 124 / 116; 3600 -> 2048 at 4096 161 / 169, -> 1500 126 / 130).
// An eighth more workgroups than units is not beyond one round yet: 16 x 64 tiles of the small kernel run two to a unit (whole int8 forwards, grid / XCD:
// 1296 -> 128 at 2176, 272 workgroups, 29.5 / 30.0, 1936 -> 256 at 1152, 288, 15.5 / 16.3; 128 x 64 tiles 124.9 / 123.8, 3136 -> 576 at 4096, 288).
// All states of one group of features before the next, whose weights are then fetched once: no faster than the grid's order at the
// small batches where weights are the larger part, 160 states 16.6 -> 17.1.
bool by_xcd(const GemmParams& p, dim3 grid) {
    const bool l2 = (int64_t)p.n_tiles * p.k_steps * 1024 <= 4 << 20;
    return grid.y > 1 && ((grid.x & 7) != 0 || (l2 && (int64_t)grid.x * grid.y > most_groups()));
}

template <int EL, int EPI, int RT, int NT>
hipError_t go(const GemmParams& q, hipStream_t s) {
    GemmParams p = q;
    const dim3 grid((unsigned)((p.B + 16 * RT - 1) / (16 * RT)), (unsigned)((p.n_tiles + NT - 1) / NT));
    p.by_xcd = by_xcd(q, grid);
#define GO(RELU, FRAG, XH) gemm_ksplit_kernel<EL, EPI, RT, NT, RELU, FRAG, XH><<<grid, dim3(64 * KS_W), 0, s>>>(p)
#define GO2(RELU, FRAG) do { if (p.xh) GO(RELU, FRAG, true); else GO(RELU, FRAG, false); } while (0)
    if (p.x_frag) { if (p.relu_in) GO2(true, true); else GO2(false, true); return hipGetLastError(); }
    if (p.relu_in) GO2(true, false);
    else GO2(false, false);
#undef GO2
#undef GO
    return hipGetLastError();
}

// The same with four wavefronts on 16 states x 64 features of row-major int8: wavefront w takes the steps w, w + 4, ..., every
// lane fetches its fragment's 16 bytes itself and wavefront t finishes feature tile t.  Shorter than the kernel above (no turn
// through LDS, half the partial sums), it is the faster one for narrow layers at middle batches: see ksplit_small_i8.
constexpr int KM_W = 4, KM_NT = 4;
template <bool XH>
__global__ __launch_bounds__(64 * KM_W) void gemm_ksplit_small_i8_kernel(const GemmParams p) {
    __shared__ __attribute__((aligned(16))) v4i s_part[KM_W * KM_NT * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const GemmTile tile = gemm_tile<!XH>(p.by_xcd);
    const int64_t b = (int64_t)tile.x * 16 + j;
    const int nt0 = tile.y * KM_NT, nts = min(p.n_tiles - nt0, KM_NT);
    const char* row = (const char*)p.x + min(b, p.B - 1) * p.Kp_bytes;      // states past the batch re-read the last one
    LstmState<XH, 64 * KM_W, 16> lstm(p, (int64_t)tile.x * 16, tile.y, tid);

    v4i acc[KM_NT];
#pragma unroll
    for (int t = 0; t < KM_NT; ++t) acc[t] = (v4i){0, 0, 0, 0};
    auto load = [&](int st, v4i (&a)[KM_NT], v4i& x) {
        const int sc = min(st, p.k_steps - 1);                              // past the end: a valid step, not multiplied
#pragma unroll
        for (int t = 0; t < KM_NT; ++t) a[t] = ((const v4i*)p.wfrag)[((int64_t)(nt0 + (t < nts ? t : 0)) * p.k_steps + sc) * 64 + lane];
        x = *(const v4i*)(row + min(sc * 64 + g * 16, (p.Kp_bytes - 16) & ~3));
    };
    auto mul = [&](int st, const v4i (&a)[KM_NT], v4i x) {
        if ((st + 1) * 64 > p.Kp_bytes) {                                   // the end of the row: as in the kernel above
            const int have = p.Kp_bytes - (st * 64 + g * 16);
            const int sh = have >= 16 ? 0 : have > 0 ? (16 - have) >> 2 : 4;
            const v4i v = x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int r = 0;
#pragma unroll
                for (int k = e; k < 4; ++k) r = k - e == sh ? v[k] : r;
                x[e] = r;
            }
        }
        if (p.relu_in) {
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = (int)g_relu_i8x4((uint32_t)x[e]);
        }
#pragma unroll
        for (int t = 0; t < KM_NT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t], x, acc[t], 0, 0, 0);
    };
    v4i a0[KM_NT], a1[KM_NT], x0, x1;
    load(wave, a0, x0);
    for (int st = wave; st < p.k_steps; st += 2 * KM_W) {
        load(st + KM_W, a1, x1);
        mul(st, a0, x0);
        load(st + 2 * KM_W, a0, x0);
        if (st + KM_W < p.k_steps) mul(st + KM_W, a1, x1);
    }
#pragma unroll
    for (int t = 0; t < KM_NT; ++t) s_part[(wave * KM_NT + t) * 64 + lane] = acc[t];
    __syncthreads();
    lstm.store();
    const int n0 = (nt0 + wave) * 16 + 4 * g;
    if (wave >= nts || b >= p.B || n0 >= p.Np) return;
    v4i sum = *(const v4i*)((const int*)p.bias + n0);
#pragma unroll
    for (int w = 0; w < KM_W; ++w) sum += s_part[(w * KM_NT + wave) * 64 + lane];
    gemm_finish<EPI_REQUANT, XH>(p, sum, b, n0);
}

int64_t groups(const GemmParams& p, int rt, int nt) { return ((p.B + 16 * rt - 1) / (16 * rt)) * ((p.n_tiles + nt - 1) / nt); }

// Row-major int8 layers of at most 256 features between the batches that 16 x 32 tiles cover with one workgroup per compute
// unit and those with one 64 x 64 workgroup per two.  us, this kernel / the tile that the rule below would take (rocprofv3):
// 1936 -> 256, ReLU on the input: 600 states 4.9 / 6.0, 1000 5.1 / 5.6, 1500 7.0 / 7.6, 1800 7.0 / 8.0; 1296 -> 128: 1800 states
// 4.8 / 5.3, 3000 5.7 / 6.2, 3500 5.8 / 6.4; just beyond the 16 x 32 tiles, 1936 -> 256 at 513 5.0 / 5.4, 576 5.0 / 5.4, 1296 -> 128 at 1025 4.5 /
// 4.8, 1152 4.4 / 4.9, 3600 -> 240 at 576 6.7 / 7.2.  Smaller batches: 1936 -> 256 at 256 states 4.6 / 4.6, 512 4.6 / 4.2.  Wide layers:
// 1936 -> 2048 at 160 states 8.6 / 6.9.
bool ksplit_small_i8(const GemmParams& p) {
    return !p.x_frag && p.n_tiles <= 16 && groups(p, 1, 2) > conv_num_cus() && 2 * groups(p, 4, 4) < conv_num_cus();
}

// The smallest tile that gives at most one workgroup per compute unit.  (An eighth more were let through once; the units with a second one
// hold up the call.  us, with them / next tile: 3136 -> 512 bf16 140 states 7.7 / 7.0, 270 9.0 / 8.1, 525 11.4 / 10.1, 1100 16.1 / 12.8, 2200 24.4 /
// 19.8; 3872 -> 256 bf16 272 8.9 / 7.8, 540 12.2 / 10.2, 1100 18.1 / 15.7, 2200 25.0 / 21.8; 1296 -> 128 bf16 560 5.4 / 4.4; int8 3136 -> 512
// 140 5.4 / 5.1, 270 6.3 / 6.1, 540 7.9 / 7.5, 1100 10.6 / 9.5; 1936 -> 256 272 4.3 / 4.1, 540 5.7 / 5.4, 2200 10.8 / 10.2.)  Measured on
// 3136 -> 512 (fragment order; us, tile of states x features): bf16, 160 states 16x32 6.5, 16x16 7.2, 32x32 7.3; 500 states 32x32 7.8, 16x64 8.4, 32x64 9.8; 1000
// states 32x64 9.8, 32x32 11.4, 64x64 12.4; 2048 states 64x64 12.9, 32x64 16.1.  int8, 64
// states 16x16 4.0, 16x32 4.3; 160 states 16x32 4.3, 16x16 4.5; 512 states 32x32 5.7, 16x64 6.2, 16x32 6.6; 1000 states 32x64 7.2,
// 32x32 8.4; 2048 states 64x64 9.2, 32x64 10.8.  bf16 beyond one 64x64 workgroup per unit: 128x64, half the fetches of the weights (3136 -> 512
// in fragment order, this kernel alone, 64x64 / 128x64: 2100 states 23.0 / 18.7, 3000 23.6 / 18.1, 4096 23.7 / 18.7, 8192 45.6 / 35.2;
// whole forwards with row-major states, 3872 -> 256 at 5000 706 / 695, 6500 898 / 889, 8192 1107 / 1101).
template <int EL, int EPI>
hipError_t pick(const GemmParams& p, hipStream_t s) {
    const int64_t most = conv_num_cus();
    if (groups(p, 1, 1) <= most) return go<EL, EPI, 1, 1>(p, s);
    if (groups(p, 1, 2) <= most) return go<EL, EPI, 1, 2>(p, s);
    if constexpr (EL == EL_I8) {
        if (ksplit_small_i8(p)) {
            const dim3 grid((unsigned)((p.B + 15) / 16), (unsigned)((p.n_tiles + KM_NT - 1) / KM_NT));
            GemmParams q = p;
            q.by_xcd = by_xcd(p, grid);
            if (p.xh) gemm_ksplit_small_i8_kernel<true><<<grid, dim3(64 * KM_W), 0, s>>>(q);
            else gemm_ksplit_small_i8_kernel<false><<<grid, dim3(64 * KM_W), 0, s>>>(q);
            return hipGetLastError();
        }
    }
    if (groups(p, 2, 2) <= most) return go<EL, EPI, 2, 2>(p, s);
    if (groups(p, 2, 4) <= most) return go<EL, EPI, 2, 4>(p, s);
    if constexpr (EL == EL_BF16) { if (groups(p, 4, 4) > most) return go<EL, EPI, 8, 4>(p, s); }
    return go<EL, EPI, 4, 4>(p, s);
}

}  // namespace

// int8 layers only up to one 64 x 64 workgroup per compute unit: beyond that the kernels that share the weights through LDS are
// faster (us, this / theirs: 3136 -> 2048 at 575 states, 288 workgroups, 21.4 / 18.2; 1936 -> 2048 there 19.3 / 16.3; at 256
// workgroups 3136 -> 512 9.2 / 9.6, 1936 -> 256 10.4 / 14.1, 1296 -> 128 at 8192 states 9.1 / 9.5).  Where the weights exceed the
// 4 MB of an XCD's second-level cache, the streaming kernel is as fast from an eighth more 32 x 64 tiles than compute units on (3136 -> 2048:
// 160 states, 32 x 64 tiles, 8.0 / 10.4; 257, 64 x 64 tiles from here on, 9.9 / 10.3, 288 10.0 / 10.2, 300 10.9 / 10.6, 400 12.5 / 12.2, 500 13.6 /
// 13.2; -> 1536: 321 9.7 / 9.9, 384 9.9 / 10.1; -> 1344: 385 9.9 / 10.6, 416 9.9 / 11.3).
// bf16 layers beyond one 64 x 64 workgroup per compute unit (128 x 64 tiles) stay here while the eighth of K that a wavefront walks is at
// least eight steps (1296 -> 128 at 10000 20.5 / 16.5), five and a half up to an eighth more than one workgroup (900 -> 512, 28 steps of K, at 2049
// states 14.1 / 12.0, 2304 13.6 / 12.3; 1296 -> 128, 41, at 8193 16.6 / 14.8, 9216 17.9 / 15.2; 1452 -> 256, 46, at 4097 19.0 / 20.8, 4608 18.4 / 19.7;
// 1568 -> 256, 49, 16.9 / 21.2, 16.8 / 21.0; 1800 -> 256, 57, 21.7 / 23.7, 21.2 / 23.0; 1936 -> 256, 61, 21.8 / 25.3, 21.0 / 24.1), and the rounds of
// workgroups are full enough.  States in fragment order: one round, or
// weights of at most 8 MB (us, this / gemm_kernel: 3136 -> 512 at 3000 states 18.1 / 28.3, 4096 18.7 / 27.1, 4500, two rounds, 33.9 / 42.5, 6000
// 35.2 / 38.9, 12000 52.6 / 77.0; 2304 -> 512 at 4500 27.8 / 31.7, 6000 28.9 / 28.3; 3136 -> 1024 at 2100 34.5 / 34.6, 4096 36.0 / 42.7), or 85 %
// of the rounds (3136 -> 2048 at 1050, 56 %, 37.9 / 35.3, 3300, 81 %, 79.1 / 71.5, 2600 60.7 / 82.0, 4096 69.2 / 80.1).  Row-major states:
// up to four rounds, the last one full (3872 -> 256 at 5000 31 / 49, 8192 40 / 51, 9300 85 / 60; 3872 -> 2048 at 2000, two rounds, 62 / 82,
// 4096, four, 121 / 151; 6000, six, 313 / 243).
bool gemm_ksplit_supported(const GemmParams& p, Elem el, GemmEpi epi) {
    if (p.B <= 0 || p.k_steps < KSPLIT_PARTS) return false;
    const int64_t cus = conv_num_cus();
    if (el == EL_BF16) {
        if (epi != EPI_BF16) return false;
        if (groups(p, 4, 4) <= cus) return true;
        const int64_t g = groups(p, 8, 4), rounds = (g + cus - 1) / cus;
        if (2 * p.k_steps < (groups(p, 4, 4) <= most_groups() ? 11 : 16) * KSPLIT_PARTS) return false;
        if (rounds == 1) return true;
        if (!p.x_frag) return rounds <= 4 && 10 * g >= 9 * rounds * cus;
        return (int64_t)p.n_tiles * p.k_steps * 1024 <= 8 << 20 || 20 * g >= 17 * rounds * cus;
    }
    if (epi != EPI_REQUANT || groups(p, 4, 4) > cus) return false;
    return (int64_t)p.n_tiles * p.k_steps * 1024 <= 4 << 20 || groups(p, 2, 4) <= most_groups() || !gemm_stream_supported(p);
}

hipError_t launch_gemm_ksplit(const GemmParams& p, Elem el, hipStream_t s) {
    return el == EL_I8 ? pick<EL_I8, EPI_REQUANT>(p, s) : pick<EL_BF16, EPI_BF16>(p, s);
}

}  // namespace accerl
