// SGAT activation transform (Eq. 11) for calls whose 64 x 128 tiles leave CUs
// idle: x'_i = x_i P G_{s_i} with the k chunks of one output split over the
// waves of a workgroup.
//
// The fixed order (transform.hip) is a chain of fused multiply-adds inside each
// chunk of 256 k, and an ascending sum of the chunk totals.  The chunks are
// therefore independent until that sum: wave w of W takes chunks w, w + W, ...,
// each from a zeroed accumulator on v_mfma_f32_16x16x4_f32 as in the tiled
// kernel, W chunk totals meet in LDS, and are added there in ascending order to
// a running total that starts at +0.  Every result is bit for bit the tiled
// kernel's.
//
// What bounds it: reading P (4 K^2 bytes) up to about 32 rows, the fp32 matrix
// cores above.  The tiled kernel has ceil(K / 128) workgroups per 64 rows and
// each walks all of K (32 workgroups at K = 4096), so a decode-sized call read
// P at 0.3 TB/s.  Here a workgroup owns RB x CB blocks of 16 x 16 outputs and
// holds up to 16 waves; no operand is shared between waves (each has its own
// k), so both go straight from memory into registers, two batches of 32 k in
// flight per wave: P as CB consecutive columns per lane (1 KB per load at CB =
// 4; the 16 columns of MFMA j are CB i + j), X as the 8 fp16 of k 8 kl .. + 7
// per lane, moved to the MFMA's k slots across the four 16-lane rows.  (Four
// batches in flight were no faster: 22.0 against 21.5 us at 16 x 4096.)
// 16 rows, time (against 32 x 256 tiles walking all of K): K = 512 4.6 us
// (30.9), 4096 21.5 (226; P alone takes 13.7 at the copy rate), 12288 127 (687;
// 123), 18944 335 (1060; 293).  64 / 128 / 256 rows at K = 4096 against 64 x
// 128 tiles: 27 / 39 / 74 us (167 / 166 / 166).
#include "tile_common.hpp"
#include "transform_plan.hpp"

namespace sq {
namespace {

static_assert(kChunk == kSplitChunk, "the rule counts chunks of the fixed order");

typedef float f32x4 __attribute__((ext_vector_type(4)));

// CB consecutive fp32 of P per lane
template <int CB>
struct Vec;
template <>
struct Vec<1> { typedef float T; };
template <>
struct Vec<2> { typedef float T __attribute__((ext_vector_type(2))); };
template <>
struct Vec<4> { typedef f32x4 T; };

__device__ __forceinline__ float load_p(const __amdgpu_buffer_rsrc_t& r, int voff, int soff, Vec<1>::T*) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ Vec<2>::T load_p(const __amdgpu_buffer_rsrc_t& r, int voff, int soff, Vec<2>::T*) {
    return __builtin_bit_cast(Vec<2>::T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
__device__ __forceinline__ Vec<4>::T load_p(const __amdgpu_buffer_rsrc_t& r, int voff, int soff, Vec<4>::T*) {
    return __builtin_bit_cast(Vec<4>::T, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ float elem(const float& v, int) { return v; }
template <typename V>
__device__ __forceinline__ float elem(const V& v, int i) { return v[i]; }

// Workgroup barrier for LDS only: this wave's LDS accesses are complete, its
// loads from memory stay in flight (the fence of __syncthreads would drain them).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int RB, int CB>
__global__ __launch_bounds__(split_waves(RB * CB) * kWave) void transform_split_kernel(const uint16_t* __restrict__ X,
                                                             const uint8_t* __restrict__ state,
                                                             const float* __restrict__ P, int M, int K, int dm, int du,
                                                             float* __restrict__ Xp) {
    typedef typename Vec<CB>::T V;
    constexpr int BM = 16 * RB, BN = 16 * CB;
    constexpr int U = 8;                             // k quads per batch: the 32 k of one X load
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    V* red = reinterpret_cast<V*>(smem);             // [wave][row block][result register][lane]
    const int tid = threadIdx.x;
    const int W = blockDim.x / kWave;
    const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    V* tot = red + W * RB * 4 * kWave;               // [row block][result register][lane]
    int rt, ct;
    const int R = (M + BM - 1) / BM;
    xcd_tile(blockIdx.x, R, K / BN, R, rt, ct);
    const int row0 = rt * BM, col0 = ct * BN;
    const int kl = lane / 16, il = lane % 16;

    const int pv = (kl * K + col0 + CB * il) * 4;    // this lane's P offset within four k rows
    int xv[RB];                                      // this lane's X row offset
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int r = row0 + 16 * i + il;
        xv[i] = r < M ? r * K * 2 + 16 * kl : (int)kOOB;
    }

    const int nch = (K + kChunk - 1) / kChunk;
    struct Batch {
        V p[U];
        v4i x[RB];
    };
    Batch b0, b1;
    auto load = [&](Batch& b, const __amdgpu_buffer_rsrc_t& rP, const __amdgpu_buffer_rsrc_t& rX, int q0) {
#pragma unroll
        for (int q = 0; q < U; ++q) b.p[q] = load_p(rP, pv, (q0 + q) * 16 * K, (V*)nullptr);
#pragma unroll
        for (int i = 0; i < RB; ++i) b.x[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, xv[i], q0 * 8, 0);
    };
    f32x4 acc[RB][CB];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;
    };
    auto compute = [&](const Batch& b) {
        uint32_t x[RB][4];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            x[i][0] = __builtin_amdgcn_perm((uint32_t)b.x[i].z, (uint32_t)b.x[i].x, 0x05040100u);
            x[i][1] = __builtin_amdgcn_perm((uint32_t)b.x[i].z, (uint32_t)b.x[i].x, 0x07060302u);
            x[i][2] = __builtin_amdgcn_perm((uint32_t)b.x[i].w, (uint32_t)b.x[i].y, 0x05040100u);
            x[i][3] = __builtin_amdgcn_perm((uint32_t)b.x[i].w, (uint32_t)b.x[i].y, 0x07060302u);
            transpose_rows4(x[i][0], x[i][1], x[i][2], x[i][3]);
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const float a = q % 2 ? hi_h(x[i][q / 2]) : lo_h(x[i][q / 2]);
#pragma unroll
                for (int j = 0; j < CB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, elem(b.p[q], j), acc[i][j], 0, 0, 0);
            }
        }
    };
    auto rsrc_p = [&](int c) {
        const int n = c < nch ? min(kChunk, K - c * kChunk) : 0;
        return make_rsrc(P + (size_t)(c < nch ? c : 0) * kChunk * K, (uint32_t)n * K * 4);
    };
    auto rsrc_x = [&](int c) {
        return make_rsrc(X + (c < nch ? c : 0) * kChunk, c < nch ? (uint32_t)(M * K - c * kChunk) * 2 : 0u);
    };

    __amdgpu_buffer_rsrc_t rP = rsrc_p(wave), rX = rsrc_x(wave);
    load(b0, rP, rX, 0);
    for (int c0 = 0; c0 < nch; c0 += W) {            // W chunks at a time, one per wave
        const int c = c0 + wave;
        const int nq = c < nch ? min(kChunk, K - c * kChunk) / 4 : 0;   // a multiple of 16 = 2 U
        clear();
        for (int q = 0; q < nq; q += 2 * U) {
            load(b1, rP, rX, q + U);
            __builtin_amdgcn_sched_barrier(0);
            compute(b0);
            __builtin_amdgcn_sched_barrier(0);
            const bool more = q + 2 * U < nq;        // else the wave's next chunk (zeros past the last)
            if (!more) {
                rP = rsrc_p(c + W);
                rX = rsrc_x(c + W);
            }
            load(b0, rP, rX, more ? q + 2 * U : 0);
            __builtin_amdgcn_sched_barrier(0);
            compute(b1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (c < nch) {
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    V t;
                    if constexpr (CB == 1) {
                        t = acc[i][0][v];
                    } else {
#pragma unroll
                        for (int j = 0; j < CB; ++j) t[j] = acc[i][j][v];
                    }
                    red[((wave * RB + i) * 4 + v) * kWave + lane] = t;
                }
        }
        lds_barrier();                               // chunk totals written
        const int nv = min(W, nch - c0);
        for (int u = wave; u < RB * 4; u += W) {
            V t;
            if (c0 > 0) {
                t = tot[u * kWave + lane];
            } else {
                if constexpr (CB == 1) {
                    t = 0.0f;
                } else {
#pragma unroll
                    for (int j = 0; j < CB; ++j) t[j] = 0.0f;
                }
            }
            for (int w = 0; w < nv; ++w) t = t + red[(w * RB * 4 + u) * kWave + lane];
            if (c0 + W < nch) {
                tot[u * kWave + lane] = t;
                continue;
            }
            const int r = row0 + 16 * (u / 4) + 4 * kl + u % 4;
            if (r >= M) continue;
            if (state) {
                const bool masked = state[r] != 0;
                if constexpr (CB == 1) {
                    t = kept(col0 + il, K, dm, du, masked) ? t : 0.0f;
                } else {
#pragma unroll
                    for (int j = 0; j < CB; ++j) t[j] = kept(col0 + CB * il + j, K, dm, du, masked) ? t[j] : 0.0f;
                }
            }
            *reinterpret_cast<V*>(Xp + (size_t)r * K + col0 + CB * il) = t;
        }
        lds_barrier();                               // and read, before the next are written
    }
}

template <int RB, int CB>
hipError_t launch_split(const uint16_t* X, const uint8_t* state, const float* P, int M, int K, int dm, int du, int W,
                        float* Xp, hipStream_t st) {
    constexpr int NW = split_waves(RB * CB);
    constexpr int kSlot = RB * CB * 1024;            // LDS bytes of one wave's chunk totals
    static std::atomic<int> lds_set[kMaxDevices];
    const hipError_t attr = allow_dynamic_lds(reinterpret_cast<const void*>(&transform_split_kernel<RB, CB>),
                                              (NW + 1) * kSlot, lds_set);
    if (attr != hipSuccess) return attr;
    const unsigned grid = (unsigned)((M + 16 * RB - 1) / (16 * RB) * (K / (16 * CB)));
    hipLaunchKernelGGL((transform_split_kernel<RB, CB>), dim3(grid), dim3(W * kWave), (size_t)(W + 1) * kSlot, st, X,
                       state, P, M, K, dm, du, Xp);
    return hipGetLastError();
}

}  // namespace

bool transform_split_faster(int M, int K, int dm, int du, bool gated) { return split_faster(M, K, dm, du, gated); }

hipError_t launch_transform_split(const uint16_t* X, const uint8_t* state, const float* P, int M, int K, int dm,
                                  int du, float* Xp, hipStream_t st) {
    const SplitShape s = split_shape(M, K);
    if (s.rb == 4) return launch_split<4, 4>(X, state, P, M, K, dm, du, s.waves, Xp, st);
    if (s.rb == 2) return launch_split<2, 4>(X, state, P, M, K, dm, du, s.waves, Xp, st);
    if (s.cb == 4) return launch_split<1, 4>(X, state, P, M, K, dm, du, s.waves, Xp, st);
    if (s.cb == 2) return launch_split<1, 2>(X, state, P, M, K, dm, du, s.waves, Xp, st);
    return launch_split<1, 1>(X, state, P, M, K, dm, du, s.waves, Xp, st);
}

}  // namespace sq
