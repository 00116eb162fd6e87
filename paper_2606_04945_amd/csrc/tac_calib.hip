// TAC closed-form calibration (Sec. 3.3 closed-form estimation; App. C).
//
// From paired attention outputs Z_fp (quantisers off) and Z_q (quantisers on),
// fp16 [N][C], per block of g channels:
//   mu_b    = (1/N) sum_i z_i,   Sigma_b = (1/N) sum_i z_i z_i^T - mu_b mu_b^T   (both passes)
//   lambda  = rho max(Tr(Sigma_q) / g, eps)
//   M       = Sigma_fp^(1/2) (Sigma_q + lambda I)^(-1/2),  A^p = Q diag(max(l_i, 1e-12)^p) Q^T
//   M_sv    = U diag((1 - eta) sigma + eta mean(sigma)) V^T,  M = U diag(sigma) V^T
//   M_final = (1 - alpha) M_sv + alpha I,   d = mu_fp - M_final mu_q
// stored as fp16 (one round-to-nearest-even from fp64) in the layout the TAC
// kernels read, tac_M [C/g][g][g] (row r, column c) and tac_d [C].
//
// Three kernels, all arithmetic in fp64:
//  * tac_stats_kernel: second moments and sums of both inputs, per chunk of
//    tokens, on the fp64 matrix cores.
//  * tac_power_kernel, one workgroup per block and input: adds the chunk
//    partials in chunk order, forms the covariance and its power +1/2 or -1/2.
//  * tac_match_kernel, one workgroup per block: the product of the powers, its
//    singular value decomposition, smoothing, shrinkage, bias and outputs.
// Both decompositions are one-sided (Hestenes) Jacobi, jacobi_columns below.
// Results depend only on the inputs (every sum has a fixed order); they agree
// with an fp64 LAPACK evaluation to rounding, not bit for bit.
#include "sq_internal.hpp"

namespace sq {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxChunks = 64;
constexpr int kChunkTok = 128;          // tokens per chunk before the caps
constexpr double kEigFloor = 1e-12;

// ----------------------------------------------------------------- statistics

// part layout: [pass][chunk][block][g*g second moments, then g sums]
//
// A workgroup takes a span of S channels (whole blocks) and a chunk of tokens,
// stages 64 or 32 tokens at a time in LDS (the next tile's loads in flight
// meanwhile) and multiplies 16 x 16 channel tiles with v_mfma_f64_16x16x4_f64,
// four tokens at a time: lane l supplies z[token l / 16][channel l % 16] of
// both tiles, so the only operand work is two conversions.  A block of g > 16 is
// symmetric: only its upper tiles are computed and stored.  Blocks of g < 16
// are read off the diagonal of one tile.
// Bound by HBM and the fp64 matrix cores about alike at g = 16: 8192 x 4096
// pairs are 134 MB (27 us at the copy rate) and 2.1 Gflop in whole tiles (29 us
// at the 73 TFLOP/s the instruction reaches); 46 us.  Vector FMAs over tiles
// staged as fp64 took 184 us, with four times the partial sums.
template <int G>
struct StatsShape {
    static constexpr int S = G > 64 ? G : 64;             // channels per workgroup
    static constexpr int NT = G > 64 ? 512 : 256;         // threads
    static constexpr int BT = G > 16 ? G / 16 : 1;        // 16-channel tiles a block spans
    static constexpr int PER = BT * (BT + 1) / 2;         // upper tiles of a block (of one tile for g <= 16)
    static constexpr int JOBS = S / (16 * BT) * PER;
    static constexpr int WAVES = NT / kWave;
    static constexpr int JPW = (JOBS + WAVES - 1) / WAVES;
};
constexpr int kTileTok = 64;            // tokens per tile (chunks are whole tiles)

// A tile's element in LDS: blocks of g > 16 use each channel BT + 1 times, so they
// are widened once, as they are staged.
template <int G>
struct StatsElem { typedef double T; };
template <>
struct StatsElem<1> { typedef uint16_t T; };
template <>
struct StatsElem<2> { typedef uint16_t T; };
template <>
struct StatsElem<4> { typedef uint16_t T; };
template <>
struct StatsElem<8> { typedef uint16_t T; };
template <>
struct StatsElem<16> { typedef uint16_t T; };
__device__ __forceinline__ double widen(uint16_t h) { return (double)h2f(h); }
__device__ __forceinline__ double widen(double v) { return v; }

template <int G>
__global__ __launch_bounds__(StatsShape<G>::NT) void tac_stats_kernel(const uint16_t* __restrict__ Zf,
                                                                     const uint16_t* __restrict__ Zq, int N, int C,
                                                                     int tok_per_chunk, int chunks,
                                                                     double* __restrict__ part) {
    using Sh = StatsShape<G>;
    constexpr int S = Sh::S, NT = Sh::NT, JPW = Sh::JPW;
    typedef typename StatsElem<G>::T E;
    constexpr bool WIDE = sizeof(E) == 8;
    constexpr int LD = S + (WIDE ? 0 : 16);              // fp16 rows: four tokens on different banks
    constexpr int TOK = WIDE ? kTileTok / 2 : kTileTok;  // tokens staged at a time
    constexpr int VPT = TOK * S / 8 / NT;                // 16-byte loads per thread per tile
    static_assert(VPT * 8 * NT == TOK * S, "tile split");
    __shared__ __attribute__((aligned(16))) E tile[TOK * LD];

    const int tid = threadIdx.x;
    const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int c0 = blockIdx.x * S;
    const int chunk = blockIdx.y, pass = blockIdx.z;
    const uint16_t* Z = pass == 0 ? Zf : Zq;
    const int t0 = chunk * tok_per_chunk;
    const int t1 = min(N, t0 + tok_per_chunk);
    const int il = lane % 16, kl = lane / 16;

    int ta[JPW], tb[JPW];                                // channel tiles of this wave's jobs
#pragma unroll
    for (int w = 0; w < JPW; ++w) {
        const int job = wave + w * Sh::WAVES;
        int u = job % Sh::PER, a = 0;
        while (u >= Sh::BT - a) u -= Sh::BT - a, ++a;    // u-th upper tile of the block: row a, column a + u
        const int base = job / Sh::PER * Sh::BT;
        ta[w] = base + a;
        tb[w] = base + a + u;
    }

    uint4 raw[VPT];
    auto fetch = [&](int tb0) {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int e = (tid + v * NT) * 8;
            const int t = tb0 + e / S;
            raw[v] = make_uint4(0, 0, 0, 0);             // tokens past t1 contribute zeros
            if (t < t1) raw[v] = *reinterpret_cast<const uint4*>(Z + (size_t)t * C + c0 + e % S);
        }
    };
    f64x4 acc[JPW];
    double sum[JPW];
#pragma unroll
    for (int w = 0; w < JPW; ++w) acc[w] = f64x4{0.0, 0.0, 0.0, 0.0}, sum[w] = 0.0;

    fetch(t0);
    for (int tk = t0; tk < t1; tk += TOK) {
#pragma unroll
        for (int v = 0; v < VPT; ++v) {
            const int e = (tid + v * NT) * 8;
            E* dst = tile + e / S * LD + e % S;
            if constexpr (WIDE) {
                const uint16_t* h = reinterpret_cast<const uint16_t*>(&raw[v]);
#pragma unroll
                for (int q = 0; q < 8; ++q) dst[q] = widen(h[q]);
            } else {
                *reinterpret_cast<uint4*>(dst) = raw[v];
            }
        }
        __syncthreads();
        if (tk + TOK < t1) fetch(tk + TOK);
#pragma unroll 4
        for (int k = 0; k < TOK; k += 4) {
            const E* row = tile + (k + kl) * LD + il;
#pragma unroll
            for (int w = 0; w < JPW; ++w) {
                if (JPW * Sh::WAVES > Sh::JOBS && wave + w * Sh::WAVES >= Sh::JOBS) break;
                const double a = widen(row[16 * ta[w]]);
                const double b = Sh::BT == 1 ? a : widen(row[16 * tb[w]]);
                acc[w] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[w], 0, 0, 0);
                sum[w] += a;
            }
        }
        __syncthreads();
    }
    const size_t stride = (size_t)G * G + G;
    double* base = part + ((size_t)pass * chunks + chunk) * (C / G) * stride;
#pragma unroll
    for (int w = 0; w < JPW; ++w) {
        if (wave + w * Sh::WAVES >= Sh::JOBS) break;
        const int ca = c0 + 16 * ta[w], cb = c0 + 16 * tb[w];   // first channels of the two tiles
        const int col = cb + il;
#pragma unroll
        for (int v = 0; v < 4; ++v) {                    // result register v: row 4 v + l / 16, column l % 16
            const int row = ca + 4 * v + kl;
            if (row / G == col / G) base[(size_t)(row / G) * stride + row % G * G + col % G] = acc[w][v];
        }
        double t = sum[w];                               // the four token slots of a channel
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        if (ta[w] == tb[w] && kl == 0) base[(size_t)(col / G) * stride + (size_t)G * G + col % G] = t;
    }
}

// ----------------------------------------------------------------- closed form

// One RNE rounding of an fp64 value to fp16 bits (overflow to infinity).
__device__ uint16_t f64_to_f16(double x) {
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint16_t sign = (uint16_t)((b >> 48) & 0x8000u);
    const int e = (int)((b >> 52) & 0x7FF);
    const uint64_t frac = b & 0xFFFFFFFFFFFFFull;
    if (e == 0x7FF) return sign | 0x7C00u | (frac ? 0x200u : 0u);
    if (e == 0) return sign;                              // zero or an fp64 subnormal
    const uint64_t mant = frac | (1ull << 52);            // value = mant * 2^(E - 52)
    int E = e - 1023;
    int shift;                                            // bits dropped from mant
    if (E >= -14) {
        shift = 42;                                       // keep 11 bits (implicit one + 10)
    } else {
        shift = 28 - E;                                   // subnormal: units of 2^-24
        if (shift > 60) return sign;                      // below half the smallest subnormal
    }
    uint64_t q = mant >> shift;
    const uint64_t rem = mant & ((1ull << shift) - 1);
    const uint64_t half = 1ull << (shift - 1);
    if (rem > half || (rem == half && (q & 1))) ++q;
    if (E >= -14) {
        if (q == (1ull << 11)) {                          // mantissa carried into the exponent
            q >>= 1;
            ++E;
        }
        if (E > 15) return sign | 0x7C00u;
        return sign | (uint16_t)((E + 15) << 10) | (uint16_t)(q & 0x3FFu);
    }
    return sign | (uint16_t)q;                            // q == 1024 is the smallest normal
}

// Threads of the closed-form kernels: LPP lanes per pair of columns, each with
// RPT rows.
template <int G>
struct SolveShape {
    static constexpr int LPP = G >= 32 ? 16 : (G >= 8 ? 8 : G);
    static constexpr int RPT = G / LPP;
    static constexpr int H = G / 2;                       // pairs per round
    static constexpr int NT = H * LPP < kWave ? kWave : H * LPP;
    static constexpr bool VREG = G > 64;                  // V in registers: W alone fills the LDS
    static constexpr int LDS_POWER = (VREG ? 1 : 2) * G * G * 8;
    static constexpr int LDS_MATCH = (VREG ? 1 : 3) * G * G * 8;   // and M_final
};

// Orders this workgroup's LDS accesses.  One wave's are performed in order, so
// there only the compiler has to keep them so.
template <int NT>
__device__ __forceinline__ void sync() {
    if (NT > kWave) {
        __syncthreads();
    } else {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    }
}

// The value of the lane that a DPP control selects.
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)u, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// Sum over L consecutive lanes (L a power of two up to 16, aligned), in every lane.
template <int L>
__device__ __forceinline__ double lanes_sum(double x) {
    if (L >= 2) x += dpp<0xB1>(x);                        // quad_perm [1, 0, 3, 2]
    if (L >= 4) x += dpp<0x4E>(x);                        // quad_perm [2, 3, 0, 1]
    if (L >= 8) x += dpp<0x141>(x);                       // row_half_mirror: the other quad of eight
    if (L >= 16) x += dpp<0x140>(x);                      // row_mirror: the other eight of sixteen
    return x;
}

// 1 / sqrt(a) to working precision for a in [1, 2]: v_rsq_f64 (4e-8 off) and two
// Newton steps.  (One third-order step is shorter, but c^2 + s^2 then drifts over
// the rotations: 3.8e-15 against 1.5e-15 from LAPACK at G = 16, 4.1e-14 against
// 3.9e-15 at 128.)
__device__ __forceinline__ double rsqrt_full(double a) {
    double y = __builtin_amdgcn_rsq(a);
    y = y * fma(-0.5 * a * y, y, 1.5);
    return y * fma(-0.5 * a * y, y, 1.5);
}

// What a lane met in a sweep, and whether the sweep needs another one.  A sweep
// rotates every pair to orthogonal once; what it leaves is what later rotations put
// back: a rotation by t of columns p and q gives (r, p) up to t times what (r, q)
// has.  So it is enough that no pair was farther than 2e-9 from orthogonal (far) and
// no rotation larger than 5e-8 (turned): less than 1e-16 comes back each time.  That
// is how columns of distinct norms end, whose rotations shrink with their products.
// Columns of (nearly) equal norm, from repeated eigenvalues, turn by any angle on
// rounding noise, so there every pair must be found orthogonal to working precision
// (open: farther than 4e-15; rounding leaves at most about 1e-15 at G = 128).
// Stopping at 2e-9 alone left them up to 4e-11 from LAPACK.
struct Met {
    bool far = false, open = false, turned = false;
    __device__ __forceinline__ void publish(int* flags) const {
        if (far) flags[0] = 1;
        if (open) flags[1] = 1;
        if (turned) flags[2] = 1;
    }
    __device__ __forceinline__ static bool again(const int* flags) { return flags[0] | (flags[1] & flags[2]); }
};

// The rotation (x, y) <- (c x - s y, s x + c y) that makes columns of squared
// norms al, be and product ga orthogonal: t = sign(z) / (|z| + sqrt(1 + z^2)),
// z = (be - al) / (2 ga), c = 1 / sqrt(1 + t^2), s = t c.  c and s must be
// orthonormal to working precision; t only decides how much of ga the rotation
// removes, so it is formed with the hardware's approximate reciprocal and
// reciprocal square root (a relative 1e-7 of ga is left).  `met` takes what the
// pair says about the sweep.
__device__ __forceinline__ void rotation(double al, double be, double ga, double& c, double& s, Met& met) {
    const double z = (be - al) * __builtin_amdgcn_rcp(2.0 * ga);
    const double h = fma(z, z, 1.0);
    double t = __builtin_amdgcn_rcp(fabs(z) + h * __builtin_amdgcn_rsq(h));
    t = fabs(z) < 1e100 ? copysign(t, z) : 0.5 * __builtin_amdgcn_rcp(z);   // z^2 would overflow
    const double g2 = ga * ga, ab = al * be;
    t = g2 > 1e-32 * ab ? t : 0.0;                        // orthogonal already (or a zero column)
    met.far |= g2 > 4e-18 * ab;
    met.open |= g2 > 1.6e-29 * ab;
    met.turned |= fabs(t) > 5e-8;
    c = rsqrt_full(fma(t, t, 1.0));
    s = t * c;
}

// One-sided (Hestenes) Jacobi on the G columns of W in LDS (column j at j G):
// on return W holds A V for the A it came with, its columns orthogonal, and V
// (LDS, the same layout) the accumulated rotations.  For a general A that is
// U Sigma and the right singular vectors; for a symmetric positive semidefinite
// A the columns are l_j v_j, V its eigenvectors.
//
// A round works on G / 2 disjoint pairs (round-robin ordering), LPP lanes each:
// a lane reads its rows of both columns, the three products meet over the lanes
// by DPP, every lane forms the rotation itself and writes its rows back, so a
// round is one LDS round trip and one barrier (none up to G = 16, where a wave
// holds all pairs).  Sweeps end as Met says.
// Bound by the latency of a round (0.4 us at G = 16: one wave per block and
// little more than one chain of dependent fp64 instructions).  The two-sided
// form for the eigendecompositions took three passes over LDS and three
// barriers a round, with the rotations formed by a few threads by full-precision
// divides and square roots: the closed form of 256 blocks of 16 took 417 us, now
// 97; of 32 blocks of 128, 26 ms, now 4.4.
template <int G>
__device__ __forceinline__ void jacobi_columns(double* W, double* V, int* flags) {
    using Sh = SolveShape<G>;
    constexpr int NT = Sh::NT, LPP = Sh::LPP, RPT = Sh::RPT, H = Sh::H;
    const int tid = threadIdx.x;
    for (int e = tid; e < G * G; e += NT) V[e] = e / G == e % G ? 1.0 : 0.0;
    sync<NT>();
    if (G == 1) return;
    const int t = tid / LPP, j = tid % LPP;
    const bool on = t < H;                                // G < 16 leaves lanes of the wave idle
    for (int sweep = 0; sweep < 60; ++sweep) {
        if (tid < 3) flags[tid] = 0;
        sync<NT>();
        Met met;
        int a = t, b = G - 1 - t;                         // players of positions t and G - 1 - t in round 0
        for (int r = 0; r < G - 1; ++r) {
            if (on) {
                const int p = a < b ? a : b, q = a < b ? b : a;
                double x[RPT], y[RPT], vx[RPT], vy[RPT];
#pragma unroll
                for (int k = 0; k < RPT; ++k) x[k] = W[p * G + j + LPP * k], y[k] = W[q * G + j + LPP * k];
#pragma unroll
                for (int k = 0; k < RPT; ++k) vx[k] = V[p * G + j + LPP * k], vy[k] = V[q * G + j + LPP * k];
                double al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
                for (int k = 0; k < RPT; ++k) {
                    al = fma(x[k], x[k], al);
                    be = fma(y[k], y[k], be);
                    ga = fma(x[k], y[k], ga);
                }
                al = lanes_sum<LPP>(al), be = lanes_sum<LPP>(be), ga = lanes_sum<LPP>(ga);
                double c, s;
                rotation(al, be, ga, c, s, met);
#pragma unroll
                for (int k = 0; k < RPT; ++k) {
                    W[p * G + j + LPP * k] = fma(c, x[k], -s * y[k]);
                    W[q * G + j + LPP * k] = fma(c, y[k], s * x[k]);
                    V[p * G + j + LPP * k] = fma(c, vx[k], -s * vy[k]);
                    V[q * G + j + LPP * k] = fma(c, vy[k], s * vx[k]);
                }
            }
            // position 0 keeps its player; the others take the next of 1 .. G - 1
            if (t > 0) a = a == G - 1 ? 1 : a + 1;
            b = b == G - 1 ? 1 : b + 1;
            sync<NT>();
        }
        met.publish(flags);
        sync<NT>();
        const bool again = Met::again(flags);
        sync<NT>();
        if (!again) break;
    }
}

// G = 128: W alone takes 128 KB of LDS, so V lives in registers.  Eight lanes
// hold a row of V, lane j of them the positions of pairs 8 j .. 8 j + 7: index i
// of `lo` is position 8 j + i, of `hi` position G - 1 - (8 j + i).  Positions hold
// columns in round-robin order, so every round rotates lo[i] with hi[i], and
// between rounds positions 1 .. G - 1 shift by one (the two ends of a lane's run
// come from its neighbours).  After a sweep position order is column order
// again.  cs[t] holds a round's rotation of pair t, s signed so that it applies
// to (position t, position G - 1 - t).
template <int G>
__device__ __forceinline__ void jacobi_columns_vreg(double* W, double* Vout, double2* cs, int* flags) {
    using Sh = SolveShape<G>;
    constexpr int LPP = Sh::LPP, RPT = Sh::RPT;
    static_assert(Sh::NT == 8 * G && G / 16 == 8, "eight lanes per row, eight pairs each");
    const int tid = threadIdx.x;
    const int t = tid / LPP, j = tid % LPP;
    const int row = tid / 8, vj = tid % 8;
    double lo[8], hi[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        lo[i] = 8 * vj + i == row ? 1.0 : 0.0;
        hi[i] = G - 1 - (8 * vj + i) == row ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < 60; ++sweep) {
        if (tid < 3) flags[tid] = 0;
        __syncthreads();
        Met met;
        int a = t, b = G - 1 - t;
        for (int r = 0; r < G - 1; ++r) {
            const int p = a < b ? a : b, q = a < b ? b : a;
            double x[RPT], y[RPT];
#pragma unroll
            for (int k = 0; k < RPT; ++k) x[k] = W[p * G + j + LPP * k], y[k] = W[q * G + j + LPP * k];
            double al = 0.0, be = 0.0, ga = 0.0;
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                al = fma(x[k], x[k], al);
                be = fma(y[k], y[k], be);
                ga = fma(x[k], y[k], ga);
            }
            al = lanes_sum<LPP>(al), be = lanes_sum<LPP>(be), ga = lanes_sum<LPP>(ga);
            double c, s;
            rotation(al, be, ga, c, s, met);
            double2* out = cs + (r & 1) * (G / 2);        // two rounds' worth: the last round's readers may lag
            if (j == 0) out[t % 8 * 8 + t / 8] = make_double2(c, a == p ? s : -s);
#pragma unroll
            for (int k = 0; k < RPT; ++k) {
                W[p * G + j + LPP * k] = fma(c, x[k], -s * y[k]);
                W[q * G + j + LPP * k] = fma(c, y[k], s * x[k]);
            }
            if (t > 0) a = a == G - 1 ? 1 : a + 1;
            b = b == G - 1 ? 1 : b + 1;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const double2 f = out[8 * i + vj];
                const double u = lo[i], w = hi[i];
                lo[i] = fma(f.x, u, -f.y * w);
                hi[i] = fma(f.x, w, f.y * u);
            }
            // position k takes position k + 1 (1 <= k < G - 1), position G - 1 takes 1, 0 stays
            const double from_next = dpp<0x101>(lo[0]);           // row_shl:1: position 8 (vj + 1)
            const double from_prev = dpp<0x111>(hi[7]);           // row_shr:1: position G - 8 vj
            const double first = lo[1];                           // position 1 in lane 0
            const double last_lo = vj == 7 ? hi[7] : from_next;   // lane 7: position 64 follows 63
#pragma unroll
            for (int i = 0; i < 7; ++i)
                if (i > 0 || vj > 0) lo[i] = lo[i + 1];
            lo[7] = last_lo;
#pragma unroll
            for (int i = 7; i > 0; --i) hi[i] = hi[i - 1];
            hi[0] = vj == 0 ? first : from_prev;
        }
        met.publish(flags);
        __syncthreads();
        const bool again = Met::again(flags);
        __syncthreads();
        if (!again) break;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        Vout[(8 * vj + i) * G + row] = lo[i];
        Vout[(G - 1 - (8 * vj + i)) * G + row] = hi[i];
    }
    __syncthreads();
}

// out(i, j, sum_k fa(i, k) fb(k, j)) for a G x G product: 16 x 16 tiles on the
// fp64 matrix cores (k in ascending groups of four), plain sums below 16.
template <int G, int NT, typename FA, typename FB, typename OUT>
__device__ __forceinline__ void product(FA fa, FB fb, OUT out) {
    const int tid = threadIdx.x;
    if constexpr (G >= 16) {
        constexpr int T = G / 16;
        const int lane = tid % kWave, il = lane % 16, kl = lane / 16;
        for (int u = tid / kWave; u < T * T; u += NT / kWave) {
            const int i0 = u / T * 16, j0 = u % T * 16;
            f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
            for (int k = 0; k < G; k += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa(i0 + il, k + kl), fb(k + kl, j0 + il), acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) out(i0 + 4 * v + kl, j0 + il, acc[v]);
        }
    } else {
        for (int e = tid; e < G * G; e += NT) {
            double s = 0.0;
            for (int k = 0; k < G; ++k) s = fma(fa(e / G, k), fb(k, e % G), s);
            out(e / G, e % G, s);
        }
    }
}

// out(j, sum_i f(j, i)) for every column j: up to 16 lanes per column, each over
// its rows in ascending order, added in a fixed order.
template <int G, int NT, typename F, typename OUT>
__device__ __forceinline__ void column_sums(F f, OUT out) {
    constexpr int L = G < 16 ? G : 16;                    // lanes per column
    for (int e = threadIdx.x; e < (G * L + NT - 1) / NT * NT; e += NT) {
        const int j = e / L < G ? e / L : G - 1, l = e % L;
        double s = 0.0;
        for (int i = l; i < G; i += L) s += f(j, i);
        s = lanes_sum<L>(s);
        if (l == 0 && e < G * L) out(j, s);
    }
}

// Scratch of a block: the powers of the two covariances (G x G each), for G = 128
// the vectors of each pass's decomposition and M_final, and the means.
template <int G>
__device__ __forceinline__ double* block_scratch(double* wk, int b) {
    return wk + (size_t)b * (6 * G * G + 3 * G);
}

// (Sigma_fp)^(1/2) (pass 0) or (Sigma_q + lambda I)^(-1/2) (pass 1) of block
// blockIdx.x: one-sided Jacobi of the covariance, l_j = v_j . (A v_j).
template <int G>
__global__ __launch_bounds__(SolveShape<G>::NT) void tac_power_kernel(const double* __restrict__ part, int chunks,
                                                                     int N, int C, double rho, double eps,
                                                                     double* __restrict__ wk) {
    using Sh = SolveShape<G>;
    constexpr int NT = Sh::NT, GG = G * G;
    extern __shared__ __attribute__((aligned(16))) double mats[];
    __shared__ double mu[G], w[G];
    __shared__ double2 cs[Sh::VREG ? G : 1];
    __shared__ int flags[3];
    double* W = mats;
    const int tid = threadIdx.x, b = blockIdx.x, pass = blockIdx.y;
    const size_t stride = GG + G;
    const double* p0 = part + ((size_t)pass * chunks * (C / G) + b) * stride;
    const size_t step = (size_t)(C / G) * stride;         // one chunk
    double* base = block_scratch<G>(wk, b);
    double* R = base + pass * GG;
    double* Vg = base + (2 + pass) * GG;
    double* V = Sh::VREG ? Vg : mats + GG;

    auto chunk_sum = [&](int e) {
        double s = 0.0;
#pragma unroll 8
        for (int k = 0; k < chunks; ++k) s += p0[k * step + e];
        return s / (double)N;
    };
    for (int e = tid; e < G; e += NT) {
        mu[e] = chunk_sum(GG + e);
        base[6 * GG + pass * G + e] = mu[e];
    }
    sync<NT>();
#pragma unroll 1
    for (int e = tid; e < GG; e += NT) {                  // upper tiles; the lower ones are their mirror
        const int r = e / G, c = e % G;
        if (r / 16 > c / 16) continue;
        const double v = chunk_sum(e) - mu[r] * mu[c];
        W[c * G + r] = v;
        if (r / 16 < c / 16) W[r * G + c] = v;
    }
    sync<NT>();
    if (pass == 1) {                                      // damping
        double tr = 0.0;
        for (int k = 0; k < G; ++k) tr += W[k * G + k];
        sync<NT>();
        const double lam = rho * fmax(tr / G, eps);
        for (int k = tid; k < G; k += NT) W[k * G + k] += lam;
        sync<NT>();
    }
    if constexpr (Sh::VREG)
        jacobi_columns_vreg<G>(W, V, cs, flags);
    else
        jacobi_columns<G>(W, V, flags);
    column_sums<G, NT>([&](int j, int i) { return V[j * G + i] * W[j * G + i]; },
                       [&](int j, double l) {
                           l = fmax(l, kEigFloor);
                           w[j] = pass == 1 ? 1.0 / sqrt(l) : sqrt(l);
                       });
    sync<NT>();
    if constexpr (Sh::VREG) {                             // the vectors into LDS, in place of W
        for (int e = tid; e < GG; e += NT) W[e] = V[e];
        V = W;
        __syncthreads();
    }
    product<G, NT>([&](int i, int k) { return V[k * G + i] * w[k]; }, [&](int k, int j) { return V[k * G + j]; },
                   [&](int i, int j, double s) { R[j * G + i] = s; });
}

// Covariance matching, singular value smoothing, shrinkage and bias of block
// blockIdx.x from the two powers and means.
template <int G>
__global__ __launch_bounds__(SolveShape<G>::NT) void tac_match_kernel(double* __restrict__ wk, double eta,
                                                                     double alpha, uint16_t* __restrict__ tac_M,
                                                                     uint16_t* __restrict__ tac_d,
                                                                     double* __restrict__ M64,
                                                                     double* __restrict__ d64) {
    using Sh = SolveShape<G>;
    constexpr int NT = Sh::NT, GG = G * G;
    extern __shared__ __attribute__((aligned(16))) double mats[];
    __shared__ double sig[G], w[G], muq[G];
    __shared__ double2 cs[Sh::VREG ? G : 1];
    __shared__ int flags[3];
    double* W = mats;
    const int tid = threadIdx.x, b = blockIdx.x;
    double* base = block_scratch<G>(wk, b);
    const double* R1 = base;
    const double* R2 = base + GG;
    double* V = Sh::VREG ? base + 2 * GG : mats + GG;
    const double* mu = base + 6 * GG;
    for (int e = tid; e < G; e += NT) muq[e] = mu[G + e];
    product<G, NT>([&](int i, int k) { return R1[k * G + i]; }, [&](int k, int j) { return R2[j * G + k]; },
                   [&](int i, int j, double s) { W[j * G + i] = s; });
    sync<NT>();
    if constexpr (Sh::VREG)
        jacobi_columns_vreg<G>(W, V, cs, flags);
    else
        jacobi_columns<G>(W, V, flags);
    column_sums<G, NT>([&](int j, int i) { return W[j * G + i] * W[j * G + i]; },
                       [&](int j, double s) { sig[j] = sqrt(s); });
    sync<NT>();
    double sbar = 0.0;
    for (int k = 0; k < G; ++k) sbar += sig[k];
    sbar /= G;
    for (int j = tid; j < G; j += NT) {                   // factor sigma'_j / sigma_j on column j of U Sigma
        const double s = sig[j];
        w[j] = s > 0.0 ? ((1.0 - eta) * s + eta * sbar) / s : 0.0;
    }
    sync<NT>();
    double* Mf = Sh::VREG ? base + 4 * GG : mats + 2 * GG;   // M_final, with the identity shrinkage
    product<G, NT>([&](int i, int k) { return W[k * G + i] * w[k]; }, [&](int k, int j) { return V[k * G + j]; },
                   [&](int i, int j, double s) { Mf[i * G + j] = (1.0 - alpha) * s + (i == j ? alpha : 0.0); });
    sync<NT>();
    for (int e = tid; e < GG; e += NT) {
        tac_M[(size_t)b * GG + e] = f64_to_f16(Mf[e]);
        if (M64) M64[(size_t)b * GG + e] = Mf[e];
    }
    for (int r = tid; r < G; r += NT) {                   // bias
        double s = 0.0;
        for (int c = 0; c < G; ++c) s = fma(Mf[r * G + c], muq[c], s);
        const double d = mu[r] - s;
        tac_d[b * G + r] = f64_to_f16(d);
        if (d64) d64[b * G + r] = d;
    }
}

template <int G>
hipError_t launch_calib(const uint16_t* Zf, const uint16_t* Zq, int N, int C, int per, int chunks, double* part,
                        double rho, double eps, double eta, double alpha, double* wk, uint16_t* tac_M,
                        uint16_t* tac_d, double* M64, double* d64, hipStream_t st) {
    using St = StatsShape<G>;
    using Sh = SolveShape<G>;
    static std::atomic<int> power_set[kMaxDevices], match_set[kMaxDevices];
    hipError_t e = allow_dynamic_lds(reinterpret_cast<const void*>(&tac_power_kernel<G>), Sh::LDS_POWER, power_set);
    if (e != hipSuccess) return e;
    e = allow_dynamic_lds(reinterpret_cast<const void*>(&tac_match_kernel<G>), Sh::LDS_MATCH, match_set);
    if (e != hipSuccess) return e;
    const unsigned B = (unsigned)(C / G);
    hipLaunchKernelGGL(tac_stats_kernel<G>, dim3(C / St::S, chunks, 2), dim3(St::NT), 0, st, Zf, Zq, N, C, per,
                       chunks, part);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tac_power_kernel<G>, dim3(B, 2), dim3(Sh::NT), Sh::LDS_POWER, st, part, chunks, N, C, rho,
                       eps, wk);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tac_match_kernel<G>, dim3(B), dim3(Sh::NT), Sh::LDS_MATCH, st, wk, eta, alpha, tac_M, tac_d,
                       M64, d64);
    return hipGetLastError();
}

// Token chunks: about 128 tokens each, at most 64, and at most what keeps the
// partial sums under 64 MB.
void calib_plan(int N, int C, int g, int& chunks, int& per) {
    const size_t per_chunk = 2 * ((size_t)C / g) * ((size_t)g * g + g) * sizeof(double);
    const size_t cap_bytes = (size_t)64 << 20;
    int cap = (int)(cap_bytes / per_chunk);
    cap = cap < 1 ? 1 : (cap > kMaxChunks ? kMaxChunks : cap);
    chunks = (N + kChunkTok - 1) / kChunkTok;
    chunks = chunks < 1 ? 1 : (chunks > cap ? cap : chunks);
    per = (N + chunks - 1) / chunks;
    chunks = (N + per - 1) / per;
}


// The chunks that are run: as many as give about 2048 workgroups (eight per CU),
// whole tiles of tokens each, within the workspace's number.  More only add
// partial sums to write and read (64 chunks of 8192 x 4096 at g = 16: 142 MB of
// them against 134 MB of input).
void calib_chunks(int N, int C, int g, int& chunks, int& per) {
    calib_plan(N, C, g, chunks, per);
    const int spans = C / (g > 64 ? g : 64);
    const int want = (1024 + spans - 1) / spans;
    if (chunks > want) chunks = want;
    per = ((N + chunks - 1) / chunks + kTileTok - 1) / kTileTok * kTileTok;
    chunks = (N + per - 1) / per;
}

}  // namespace

size_t tac_calib_workspace_bytes(int N, int C, int g) {
    if (N <= 0 || C <= 0 || g <= 0) return 0;
    int chunks, per;
    calib_plan(N, C, g, chunks, per);
    const size_t B = (size_t)C / g, gg = (size_t)g * g;
    const size_t part = 2 * (size_t)chunks * B * (gg + g) * sizeof(double);
    const size_t work = B * (6 * gg + 3 * g) * sizeof(double);
    return ((part + 255) / 256) * 256 + work;
}

hipError_t launch_tac_calib(const uint16_t* Zf, const uint16_t* Zq, int N, int C, int g, double rho, double eps,
                            double eta, double alpha, uint16_t* tac_M, uint16_t* tac_d, double* M64, double* d64,
                            void* ws, hipStream_t st) {
    int chunks, per;
    calib_chunks(N, C, g, chunks, per);
    const size_t B = (size_t)C / g, gg = (size_t)g * g;
    double* part = static_cast<double*>(ws);
    const size_t part_bytes = 2 * (size_t)chunks * B * (gg + g) * sizeof(double);
    double* wk = reinterpret_cast<double*>(static_cast<uint8_t*>(ws) + ((part_bytes + 255) / 256) * 256);
    auto run = [&](auto launch) {
        return launch(Zf, Zq, N, C, per, chunks, part, rho, eps, eta, alpha, wk, tac_M, tac_d, M64, d64, st);
    };
    switch (g) {
        case 1: return run(launch_calib<1>);
        case 2: return run(launch_calib<2>);
        case 4: return run(launch_calib<4>);
        case 8: return run(launch_calib<8>);
        case 16: return run(launch_calib<16>);
        case 32: return run(launch_calib<32>);
        case 64: return run(launch_calib<64>);
        default: return run(launch_calib<128>);
    }
}

}  // namespace sq
