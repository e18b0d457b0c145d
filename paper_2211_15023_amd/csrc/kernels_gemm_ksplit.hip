// Dense layers whose wavefronts split K: a workgroup owns 16 * RT states x 16 * NT features, each of its eight wavefronts
// multiplies the whole tile over its own eighth of the MFMA steps with operands straight from memory, and the partial sums
// meet in LDS, where every wavefront finishes its share of the tiles.  The split of K and the order of the partial sums do
// not depend on the tile, so a state's result does not depend on the batch it is in.
//
// What bounds it: bytes in flight.  A compute unit pulls about 25 bytes per clock out of the second-level cache and the
// memory behind it however many loads its wavefronts keep open, so the tile is the smallest that still gives every unit one
// workgroup: more units pull, and none of them twice.  The kernel this replaces walked K alone in each 64 x 64 workgroup
// (64 workgroups on 256 units for 1024 states of a 3872 -> 256 layer): 42 -> 10.6 us there; 3136 -> 512 at 500 states
// 28 -> 9.7 us, at 4096 states 35 -> 27 us (rocprofv3 / HIP events less the event cost).
#include <type_traits>

#include "gemm_epilogue.h"

namespace accerl {

int conv_num_cus();   // compute units of the current device

namespace {

constexpr int KS_LDS = 64 * 1024;
constexpr int KS_W = 8;                                       // wavefronts per workgroup

template <int EL, int EPI, int RT, int NT, bool RELU, bool FRAG>
__global__ __launch_bounds__(64 * KS_W) void gemm_ksplit_kernel(const GemmParams p) {
    typedef typename std::conditional<EL == EL_I8, v4i, v4f>::type Acc;
    constexpr int W = KS_W, D = 2;                          // D steps in flight per wavefront
    constexpr int FIT = KS_LDS / (W * NT * 1024);
    constexpr int RH = RT < FIT ? RT : FIT;                   // state tiles folded at a time
    __shared__ __attribute__((aligned(16))) Acc s_part[W * RH * NT * 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int64_t b0 = (int64_t)blockIdx.x * (16 * RT);
    const int nt0 = blockIdx.y * NT;
    const int ks = p.k_steps;
    const int s0 = wave * ks / W, s1 = (wave + 1) * ks / W;   // this wavefront's steps

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
    {
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
            gemm_finish<EPI>(p, sum, b, n0);
        }
    }
}

template <int EL, int EPI, int RT, int NT>
hipError_t go(const GemmParams& p, hipStream_t s) {
    const dim3 grid((unsigned)((p.B + 16 * RT - 1) / (16 * RT)), (unsigned)((p.n_tiles + NT - 1) / NT));
#define GO(RELU, FRAG) gemm_ksplit_kernel<EL, EPI, RT, NT, RELU, FRAG><<<grid, dim3(64 * KS_W), 0, s>>>(p)
    if (p.relu_in) { if (p.x_frag) GO(true, true); else GO(true, false); }
    else { if (p.x_frag) GO(false, true); else GO(false, false); }
#undef GO
    return hipGetLastError();
}

// The smallest tile that gives at most about one workgroup per compute unit.  Measured on 3136 -> 512 bf16 (us, tile of
// states x features): 160 states 16x32 7.2, 16x16 8.6, 32x32 9.1; 500 states 32x32 9.7, 16x32 11.1, 32x64 11.5; 1000 states
// 32x64 11.9, 32x32 14.7, 64x64 15.5; 2048 states 64x64 17.8, 32x64 19.4; 4096 states 128x64 26.8, 64x64 31.5.
template <int EL, int EPI>
hipError_t pick(const GemmParams& p, hipStream_t s) {
    const int64_t most = conv_num_cus() * 9 / 8;
    auto groups = [&](int rt, int nt) { return ((p.B + 16 * rt - 1) / (16 * rt)) * ((p.n_tiles + nt - 1) / nt); };
    if (groups(1, 1) <= most) return go<EL, EPI, 1, 1>(p, s);
    if (groups(1, 2) <= most) return go<EL, EPI, 1, 2>(p, s);
    if (groups(2, 2) <= most) return go<EL, EPI, 2, 2>(p, s);
    if (groups(2, 4) <= most) return go<EL, EPI, 2, 4>(p, s);
    if constexpr (EL == EL_BF16) { if (groups(4, 4) > most) return go<EL, EPI, 8, 4>(p, s); }
    return go<EL, EPI, 4, 4>(p, s);
}

}  // namespace

// Every bf16 layer of eight steps or more.  int8 layers only up to about one 64 x 64 workgroup per compute unit: beyond that
// the kernels that share the weights through LDS are faster (3136 -> 512 at 4096 states: 12.9 us against 17.4; 1936 -> 256 at
// 8192: 17 against 20).
bool gemm_ksplit_supported(const GemmParams& p, Elem el, GemmEpi epi) {
    if (p.B <= 0 || p.k_steps < 8) return false;
    if (el == EL_BF16) return epi == EPI_BF16;
    return epi == EPI_REQUANT && ((p.B + 63) / 64) * ((p.n_tiles + 3) / 4) <= conv_num_cus() * 9 / 8;
}

hipError_t launch_gemm_ksplit(const GemmParams& p, Elem el, hipStream_t s) {
    return el == EL_I8 ? pick<EL_I8, EPI_REQUANT>(p, s) : pick<EL_BF16, EPI_BF16>(p, s);
}

}  // namespace accerl
