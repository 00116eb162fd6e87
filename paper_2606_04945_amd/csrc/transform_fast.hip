// Fast activation transform on the fp16 MFMA (x' = x P G_s, Eq. 11): the
// matrix-core alternative to the fixed-order fp32 transform.
//
// P (fp32, orthogonal, |P| <= 1) is split once, offline, into two fp16 parts of
// the scaled basis v = 2^14 P: hi = fp16(v), lo = fp16(v - hi), stored
// transposed and side by side as Ps [K][2K] (row j = column j of P: hi over k,
// then lo over k).  Then
//   2^14 x'_j = sum_k x_k hi_kj + sum_k x_k lo_kj + sum_k x_k delta_kj,
// |delta| <= 2^-22 |v| + 2^-25, and the first two sums are one fp16 GEMM of
// [x, x] (K doubled) against Ps with fp32 accumulation: the products of two
// fp16 values are exact in fp32, so the result differs from the exact x P by
// at most 2^-14 (sum_k |x_k| |delta_kj| + gamma_2K sum_k |x_k| (|hi_kj| + |lo_kj|)).
// Codes from x' match the fixed-order transform's except where a value lies
// within that bound of a rounding boundary; the fixed-order path is the one the
// codes are defined by, this one trades that for the matrix cores.
//
// The kernel is the GEMM's direct-to-LDS pipeline on fp16
// operands.  A stage holds one k step of 32 of x and the matching steps of both
// halves of Ps (hi and lo) for each k group, so x is fetched and read from LDS
// once for both: two v_mfma_f32_16x16x32_f16 per 16 x 16 tile and step (hi then
// lo, into one accumulator), the gate applied in the epilogue, fp32 out.
// What bounds it: at a thousand rows and more the fp16 matrix cores (4096 x 12288:
// 1.35 PFLOP/s executed, what a large bf16 product reaches on the card, whose clock
// falls to 1.95 GHz under this load) and the LDS reads that feed them (a 64 x 64
// wave reads 12 KB per 32 MFMAs, a 64 x 96 one 16 KB per 48, a 128 x 64 one 16 KB per
// 64); below, the latency of the k steps a wave takes one after another, which the
// k groups divide.  With a step's fragment reads and copies issued ahead of its MFMAs
// the two took turns, as one or two waves per SIMD do not cover for each other: 1024
// x 12288 629 -> 569 us with them spread between the MFMAs, 1024 x 4096 78 -> 64, 4096
// x 12288 2155 -> 1996.  Reading both halves of a cache line together where one step
// takes half of it: 4096 x 12288 1954 -> 1863, 16384 x 3584 711 -> 684.
#include "tile_common.hpp"
#include "transform_plan.hpp"

namespace sq {
namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr float kBasisScale = 16384.0f;        // 2^14
constexpr float kBasisUnscale = 1.0f / 16384.0f;

// Ps[j][k] = hi(2^14 P[k][j]), Ps[j][K + k] = lo: 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void split_basis_kernel(const float* __restrict__ P, int K,
                                                         uint16_t* __restrict__ Ps) {
    __shared__ float t[32][33];
    const int k0 = blockIdx.y * 32, j0 = blockIdx.x * 32;
    const int tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    for (int r = ty; r < 32; r += 8) t[r][tx] = P[(size_t)(k0 + r) * K + j0 + tx];
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const float v = t[tx][r] * kBasisScale;                 // element (k0 + tx, j0 + r), exact
        const uint16_t hi = f2h(v);
        const uint16_t lo = f2h(v - h2f(hi));                    // v - hi is exact in fp32
        uint16_t* row = Ps + (size_t)(j0 + r) * (2 * (size_t)K);
        row[k0 + tx] = hi;
        row[K + k0 + tx] = lo;
    }
}

// KG > 1: KG sets of WM x WN waves share the tile and take turns over its k
// steps; their sums meet in LDS.  PAIR: the copies of two steps go out together.
template <int WM, int WN, int TM, int TN, int KG, bool PAIR>
__global__ __launch_bounds__(64 * WM * WN * KG) __attribute__((amdgpu_waves_per_eu(2))) void transform_mfma_kernel(
    const uint16_t* __restrict__ X, const uint8_t* __restrict__ state, const uint16_t* __restrict__ Ps, int M, int K,
    int dm, int du, float* __restrict__ Xp) {
    constexpr int NW = WM * WN;
    constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN;
    constexpr int AB = BM * kKStep, BB = BN * kKStep;   // bytes of one stage: x, then Ps hi, then Ps lo
    constexpr int SG = AB + 2 * BB, SB = KG * SG;
    // 1 KB copies of one stage: x, then Ps hi, then Ps lo; copy q of a wave is number NW q + wave
    constexpr int CA = AB / 1024, CB = BB / 1024, CN = CA + 2 * CB, NC = CN / NW;
    static_assert(NC * NW == CN && CA % NW == 0, "stage copies must divide evenly, x and Ps apart");
    // A step takes 64 bytes of a row, half a cache line.  With k groups the two halves
    // are requested together; without, PAIR does it, for a fourth stage of LDS.
    constexpr int NS = PAIR ? 4 : 3;                     // LDS stages
    extern __shared__ __attribute__((aligned(16))) uint8_t sm[];

    const int tid = threadIdx.x;
    const int lane = tid % kWave, wave_all = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int kg = wave_all / NW, wave = wave_all % NW;
    const int wm = wave / WN, wn = wave % WN;
    int rt, ct;
    xcd_tile(blockIdx.x, (M + BM - 1) / BM, (K + BN - 1) / BN, 8, rt, ct);
    const int row0 = rt * BM, col0 = ct * BN;
    const uint32_t lda = (uint32_t)K * 2;                // X row bytes
    const uint32_t ldb = (uint32_t)K * 4;                // Ps row bytes (hi then lo)
    const int nk_all = (int)(lda / kKStep);              // k steps (each with both halves of Ps)
    const int nk = (nk_all + KG - 1) / KG;               // stages: stage kt holds steps KG kt .. KG kt + KG - 1
    const uint32_t lo_off = lda;                         // byte offset of the lo half in a Ps row
    const u32x4 rA = sgpr_rsrc(X, (uint32_t)M * lda);
    const u32x4 rB = sgpr_rsrc(Ps, (uint32_t)K * ldb);
    auto swz = [](int r) { return (r >> 1) & 3; };

    // this lane's segment of the tile's first rows; a copy takes 16 rows.  Rows past M
    // (columns past K) lie past the descriptor's end and read as zeros.
    const uint32_t seg = 16 * ((lane % 4) ^ swz(lane / 4));
    const uint32_t oa = (uint32_t)(row0 + lane / 4) * lda + seg;
    const uint32_t ob = (uint32_t)(col0 + lane / 4) * ldb + seg;
    // wave-uniform, kept apart from the vector part of an address: combined, every
    // copy's address takes a register of its own through the loop
    auto scalar = [](uint32_t o) {
        asm("" : "+s"(o));
        return o;
    };
    // copy q of this wave's share of stage skt: x, then Ps hi and lo in turn.  Past
    // the last step the descriptors are empty, so the copies bring zeros and every
    // stage has the same number of copies to wait for.
    auto copy = [&](int skt, int stage, int q) {
        const int kt = KG * skt + kg;                    // this k group's step
        const bool past = kt >= nk_all;
        const int c = q * NW + wave;
        const uint32_t lds = lds_addr(sm + stage * SB + kg * SG + c * 1024), ko = (uint32_t)kt * kKStep;
        if (q * NW < CA) {
            u32x4 r = rA;
            r[2] = past ? 0u : r[2];
            dma16(r, lds, oa + scalar(16 * c * lda + ko));
        } else {
            const int j = c - CA, lo = j >= CB;
            u32x4 r = rB;
            r[2] = past ? 0u : r[2];
            dma16(r, lds, ob + scalar(16 * (j - (lo ? CB : 0)) * ldb + (lo ? lo_off : 0) + ko));
        }
    };

    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    const int lr = lane % 16, lg = lane / 16;
    const int fo = (lg ^ swz(lr)) * 16;
    const int offA = ((wm * TM) * 16 + lr) * kKStep + fo;
    const int offB = AB + ((wn * TN) * 16 + lr) * kKStep + fo;
    // Fragments are read one stage ahead, and those reads and the copies of the stage
    // after next are spread between the MFMAs: a wave that issued them all at once
    // would wait for the queues with idle matrix cores.  The basis fragments and the
    // last two of x have a second register set; the others of x are read again into
    // the registers that their row of MFMAs has just used.
    v8h fa[2][TM], fh[2][TN], fl[2][TN];
    auto again = [](int i) { return i < TM - 2; };
    auto frag_a = [&](const uint8_t* st, int set, int i) {
        fa[again(i) ? 0 : set][i] = *reinterpret_cast<const v8h*>(st + offA + i * 16 * kKStep);
    };
    auto frag = [&](const uint8_t* st, int set, int q) {
        if (q < TN)
            fh[set][q] = *reinterpret_cast<const v8h*>(st + offB + q * 16 * kKStep);
        else if (q < 2 * TN)
            fl[set][q - TN] = *reinterpret_cast<const v8h*>(st + offB + BB + (q - TN) * 16 * kKStep);
        else
            frag_a(st, set, TM - 1 - (q - 2 * TN));
    };
    constexpr int NR = 2 * TN + (TM < 2 ? TM : 2), NM = 2 * TM * TN;
    // multiplies stage kt (register set kt % 2, LDS stage s0) while the fragments of
    // stage kt + 1 come in from s1.  The copies of stage kt + NS follow into s0; in
    // pairs, an odd step issues those of kt + 3 and kt + 4 into the two free stages.
    auto step = [&](int kt, int set, int s0, int s1) {
        constexpr int NX = NR + NC, N2 = 2 * NC;
        asm volatile("" ::: "memory");
        // stage kt + 1 has landed; this wave's reads of kt are done
        if (!PAIR)
            wait_vm<(NS - 2) * NC>();
        else if (set == 0)
            wait_vm<2 * NC>();
        else
            wait_vm<0>();
        __builtin_amdgcn_s_barrier();                    // ... and every wave's
        asm volatile("" ::: "memory");
        const uint8_t* st = sm + s1 * SB + kg * SG;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            // basis columns as the row operand: see the epilogue
            const int i = m / (2 * TN), j = m % TN;
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(m / TN % 2 ? fl[set][j] : fh[set][j],
                                                               fa[again(i) ? 0 : set][i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (again(i) && m % (2 * TN) == 2 * TN - 1) frag_a(st, set ^ 1, i);
#pragma unroll
            for (int q = m * NX / NM; q < (m + 1) * NX / NM; ++q) {
                if (q < NR)
                    frag(st, set ^ 1, q);
                else if (!PAIR)
                    copy(kt + NS, s0, q - NR);
            }
            if (PAIR && set == 1) {
#pragma unroll
                for (int q = m * N2 / NM; q < (m + 1) * N2 / NM; ++q)
                    copy(kt + 3 + q % 2, (kt + 3 + q % 2) % NS, q / 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int q = 0; q < NC; ++q) copy(s, s, q);
    wait_vm<(NS - 1) * NC>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < NR; ++q) frag(sm + kg * SG, 0, q);
#pragma unroll
    for (int i = 0; i < TM - 2; ++i) frag_a(sm + kg * SG, 0, i);
    auto next = [](int s) { return s == NS - 1 ? 0 : s + 1; };
    int s0 = 0;                                          // stage kt lives in LDS stage kt % NS
    for (int kt = 0; kt + 1 < nk; kt += 2) {
        const int s1 = next(s0), s2 = next(s1);
        step(kt, 0, s0, s1);
        step(kt + 1, 1, s1, s2);
        s0 = s2;
    }
    if (nk % 2) step(nk - 1, 0, s0, next(s0));
    wait_vm<0>();                                        // no copy outlives the loop
    auto owns = [&](int i, int j) { return KG == 1 || (i * TN + j) % KG == kg; };
    if constexpr (KG > 1) {
        // every wave is past its last fragment read: the stages take the partial
        // sums, and each group adds up and stores the blocks it owns
        static_assert((KG - 1) * NW * TM * TN * kWave * 16 <= NS * SB, "k-group partial sums fit in the stages");
        __syncthreads();
        v4f* red = reinterpret_cast<v4f*>(sm);           // [KG - 1: the groups but the owner][NW][TM][TN][lane]
        auto slot = [&](int g, int i, int j) {
            const int owner = (i * TN + j) % KG;
            return ((((g < owner ? g : g - 1) * NW + wave) * TM + i) * TN + j) * kWave + lane;
        };
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (!owns(i, j)) red[slot(kg, i, j)] = acc[i][j];
        __syncthreads();
        if (kg >= TM * TN) return;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if (!owns(i, j)) continue;
#pragma unroll
                for (int g = 0; g < KG; ++g)
                    if (g != kg) acc[i][j] += red[slot(g, i, j)];
            }
    }
    // acc[i][j]: token row lr of A block i, columns 4 lg .. 4 lg + 3 of basis block j
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int row = row0 + (wm * TM + i) * 16 + lr;
        if (row >= M) continue;
        const bool masked = state ? state[row] != 0 : false;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = col0 + (wn * TN + j) * 16 + lg * 4;
            if (col >= K || !owns(i, j)) continue;
            float4 o;
            o.x = (!state || kept(col + 0, K, dm, du, masked)) ? acc[i][j][0] * kBasisUnscale : 0.0f;
            o.y = (!state || kept(col + 1, K, dm, du, masked)) ? acc[i][j][1] * kBasisUnscale : 0.0f;
            o.z = (!state || kept(col + 2, K, dm, du, masked)) ? acc[i][j][2] * kBasisUnscale : 0.0f;
            o.w = (!state || kept(col + 3, K, dm, du, masked)) ? acc[i][j][3] * kBasisUnscale : 0.0f;
            *reinterpret_cast<float4*>(Xp + (size_t)row * K + col) = o;
        }
    }
}

}  // namespace

hipError_t launch_split_basis(const float* P, int K, uint16_t* Ps, hipStream_t st) {
    hipLaunchKernelGGL(split_basis_kernel, dim3(K / 32, K / 32), dim3(256), 0, st, P, K, Ps);
    return hipGetLastError();
}

namespace {

template <int WM, int WN, int TM, int TN, int KG, bool PAIR = KG == 1>
hipError_t launch_mfma(const uint16_t* X, const uint8_t* state, const uint16_t* Ps, int M, int K, int dm, int du,
                       float* Xp, hipStream_t st) {
    constexpr int BM = 16 * WM * TM, BN = 16 * WN * TN, LDS = (PAIR ? 4 : 3) * KG * (BM + 2 * BN) * kKStep;
    static_assert(LDS <= 160 * 1024, "the stages fit in LDS");
    const size_t tiles = (size_t)((M + BM - 1) / BM) * (size_t)((K + BN - 1) / BN);
    if (tiles > 0x7fffffffu) return hipErrorInvalidConfiguration;
    static std::atomic<int> lds_set[kMaxDevices];
    const hipError_t attr = allow_dynamic_lds(
        reinterpret_cast<const void*>(&transform_mfma_kernel<WM, WN, TM, TN, KG, PAIR>), LDS, lds_set);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((transform_mfma_kernel<WM, WN, TM, TN, KG, PAIR>), dim3((unsigned)tiles),
                       dim3(64 * WM * WN * KG), LDS, st, X, state, Ps, M, K, dm, du, Xp);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_transform_fast(const uint16_t* X, const uint8_t* state, const uint16_t* Ps, int M, int K, int dm,
                                 int du, float* Xp, hipStream_t st) {
    switch (fast_tile(M, K)) {
        case FastTile::k32x32: return launch_mfma<1, 1, 2, 2, 8>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k32x64: return launch_mfma<1, 2, 2, 2, 4>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k64x64: return launch_mfma<1, 1, 4, 4, 4>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k64x64x4: return launch_mfma<2, 2, 2, 2, 1, false>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k64x64x3: return launch_mfma<2, 2, 2, 2, 1>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k128x64: return launch_mfma<2, 1, 4, 4, 2>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k128x128: return launch_mfma<1, 2, 8, 4, 2>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k128x128x2: return launch_mfma<2, 2, 4, 4, 1, false>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k256x128: return launch_mfma<4, 2, 4, 4, 1>(X, state, Ps, M, K, dm, du, Xp, st);
        case FastTile::k256x192: return launch_mfma<4, 2, 4, 6, 1>(X, state, Ps, M, K, dm, du, Xp, st);
    }
    return hipErrorInvalidConfiguration;
}

}  // namespace sq
