// Which kernel, tile and K split a GEMM call takes: host code with no HIP in it, so
// that it is also compiled and checked without a GPU compiler.
#pragma once
#include <stddef.h>

namespace sq {
namespace {

constexpr int kKB = 64;                              // bytes per row per k step (128 4-bit / 64 8-bit codes)

// Limits of the short-M kernels that keep activations in LDS.
constexpr int kSharedMaxSteps = 32;                 // one row tile, K <= 4096: 96 KB of LDS
constexpr int kSharedMaxTileSteps = 128;            // more row tiles: row tiles x k steps <= 128 (128 KB)
constexpr int kSharedMaxWaves = 16;
constexpr size_t kFragMaxLds = 160 * 1024;

// A launch plan: tile shape and K split.
struct Plan {
    int cfg;       // 0: 256 x 128, 1: 128 x 128, 2: 64 x 64, 4: 64 x 128, 7: 128 x 256 (8-bit), 8: 128 x 128
                   // in two waves of 128 x 64 (8-bit), 9: 128 x 128 in two k groups of four waves,
                   // 10 ... 14: small grids in k groups (see choose_k_groups),
                   // 3: short M, K split in the
                   // workgroup, 5: short M, activations shared in LDS (see launch_gemm), 6: short M on
                   // fragment-ordered weights (see launch_gemm_frag)
    int bm, bn;
    int splits;    // K split count across workgroups actually used (1 = fused epilogue)
    int per;       // k steps per split
    int waves;     // cfg 3: waves sharing a column group over k; cfg 5: waves per workgroup;
                   // cfg 6: column groups per workgroup
    int kw;        // cfg 6: waves per column group, taking turns over k
    bool alds;     // cfg 6: activation fragments staged in LDS (else read from L2)
    bool whole;    // cfg 6: ... with no fewer column groups per workgroup for it
    int u, d;      // cfg 6: k steps per batch, batches in the register ring
};

Plan make_plan(int M, int N, int K, int bm, int bn, int want_splits, int bits = 4) {
    (void)M;
    (void)N;
    Plan p;
    p.cfg = -1;
    p.waves = 1;
    p.kw = 1;
    p.alds = p.whole = false;
    p.u = 2;
    p.d = 4;
    p.bm = bm;
    p.bn = bn;
    const int nk = (K * bits / 8 + kKB - 1) / kKB;
    const int s = want_splits < 1 ? 1 : (want_splits > nk ? nk : want_splits);
    p.per = (nk + s - 1) / s;
    p.splits = (nk + p.per - 1) / p.per;
    return p;
}

// Bytes of dynamic LDS the shared-activation kernel needs, 0 if it cannot run.
size_t shared_lds_bytes(int tiles, int nk) {
    if (tiles == 1) return nk <= kSharedMaxSteps ? (size_t)nk * 3 * 1024 : 0;
    return tiles * nk <= kSharedMaxTileSteps ? (size_t)tiles * nk * 1024 : 0;
}

// Dynamic LDS of the fragment-ordered short-M kernel.
size_t frag_lds_bytes(int tm, int nk, int kw, int cg, bool alds) {
    return (alds ? (size_t)tm * nk * 1024 : 0) + (kw > 1 ? (size_t)(kw - 1) * cg * tm * 1024 : 0);
}

// Small grids: tiles so small that a launch of the whole shape is at most one
// workgroup per CU, and as many k groups as their stages fit LDS, so that a CU
// still has 8 ... 16 waves and K needs no split across workgroups (its partial
// sums through HBM and the second launch cost about 4 us).  A few hundred tokens
// are bound by the latency of the k steps, not by operands or MFMAs: the time
// follows the number of steps a wave takes, so the smallest tile that still
// fits one round wins, for 4-bit and 8-bit codes alike (65 shapes, 50 ... 2000
// rows, N = 512 ... 37888, K = 1024 ... 32768, eight weights in turn, against every
// tile below and the former plans).  4-bit, former plan -> k groups: 50 x 4096 x 4096 7.7 -> 5.2 us
// (32 x 32 tiles), 64 x 12288 x 4096 12.6 -> 9.7 (64 x 64), 128 x 4096 x 12288
// 17.5 -> 14.0 (32 x 64), 250 x 4096 x 12288 25.9 -> 18.5 (64 x 64), 250 x 3584
// x 18944 37.1 -> 25.7, 512 x 4096 x 12288 37.9 -> 29.1 (64 x 128); 8-bit: 250 x
// 4096 x 4096 21.8 -> 12.6, 512 x 3584 x 18944 92 -> 68.
// Where they stand back, with the former plan's times:
//  - 32 x 32 tiles re-read the operands most; many tiles of a deep K are then
//    bound by it: 8-bit 64 x 4096 x 12288 (256 tiles, 192 k steps) 20.5 against
//    18.7 us, 4-bit 250 x 512 x 32768 (128 tiles, 256) 16.8 against 15.8, while
//    8-bit 50 x 1536 x 12288 (96, 192) takes 16.1 against 17.0;
//  - 4-bit 64 x 128 tiles of a shallow K on three quarters of the CUs or less:
//    200 x 4608 x 3584 (144 tiles) 11.7 against 11.3.
Plan choose_k_groups(int M, int N, int K, int bits) {
    const int nk = (K * bits / 8 + kKB - 1) / kKB;
    auto tiles = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    Plan none = make_plan(M, N, K, 64, 64, 1, bits);
    const struct {
        int cfg, bm, bn;
    } shapes[] = {{10, 32, 32}, {11, 32, 64}, {12, 64, 64}, {13, 64, 128}};
    for (const auto& s : shapes) {
        const long t = tiles(s.bm, s.bn);
        if (t > 256) continue;
        if (s.cfg == 10 && nk >= 160 && t * nk >= 32768) return none;
        const bool deep = nk >= 64;
        if (s.cfg == 13 && bits == 4 && !deep && t < 192) return none;
        Plan p = make_plan(M, N, K, s.bm, s.bn, 1, bits);
        // deep K: three k groups of four 64 x 32 waves (512 x 4096 x 12288 29.1
        // us) for two of four 32 x 64 (31.0; 64 x 24576 x 4096 15.3 against 14.6)
        p.cfg = s.cfg == 13 && deep ? 14 : s.cfg;
        return p;
    }
    return none;
}

// Fragment-ordered weights, few rows (from graph-replayed sweeps with rotating
// weights): at most about one workgroup per CU.  Wide layers (>= 1024 column
// groups): one wave per column group, activations in LDS; mid-width (>= 384):
// two waves per column group, activations in LDS; 257-383 groups: two waves per
// group, two groups per workgroup, activations in LDS (one group per workgroup
// would leave some CUs twice the work of the rest); up to 256: four waves per
// column group, one group per workgroup, activations from L2, a ring of two
// batches from 17 tokens on.  Batches of two k steps, or of one where that
// leaves fewer zero-weight k steps in the last pass of the ring.  At least two
// batches per wave.
Plan choose_frag_short(int M, int N, int K, int bits) {
    const int nk = (K * bits / 8 + kKB - 1) / kKB, nb = (nk + 1) / 2;
    const int groups = (N + 15) / 16, tm = (M + 15) / 16;
    Plan p = make_plan(M, N, K, 16 * tm, 16, 1, bits);
    p.cfg = 6;
    int kw, cg;
    bool alds;
    if (groups >= 1024) {
        kw = 1, cg = (groups + 255) / 256, alds = true;
    } else if (groups >= 384) {
        kw = 2, cg = tm == 1 ? (groups + 255) / 256 : (groups + 191) / 192, alds = true;
    } else if (groups > 256) {
        kw = 2, cg = 2, alds = true;
    } else {
        kw = 4, cg = 1, alds = false;
    }
    while (kw > 1 && nb < 2 * kw) kw /= 2;
    const int cg0 = cg;
    if (alds) {   // staged activations that do not fit in LDS are read from L2 instead
        cg = cg < 16 / kw ? cg : 16 / kw;
        p.whole = frag_lds_bytes(tm, nk, kw, cg, true) <= kFragMaxLds;
        while (cg > 1 && frag_lds_bytes(tm, nk, kw, cg, true) > kFragMaxLds) --cg;
        alds = frag_lds_bytes(tm, nk, kw, cg, true) <= kFragMaxLds;
    }
    if (!alds) cg = cg0 < 8 / kw ? cg0 : 8 / kw;
    p.waves = cg;
    p.kw = kw;
    p.alds = alds;
    p.d = !alds && kw == 4 && tm > 1 ? 2 : 4;
    // k steps a wave multiplies past the end: its batches rounded up to whole passes of the ring
    auto waste = [&](int u) {
        const int batches = (nk + u - 1) / u, per_wave = (batches + kw - 1) / kw;
        return (((per_wave + p.d - 1) / p.d) * p.d * kw - batches) * u;
    };
    p.u = alds && waste(1) < waste(2) ? 1 : 2;
    return p;
}

// Up to 48 rows: the kernels that stream the weights into registers, or tiles, whose
// workgroup reads a weight once for all its rows (in k groups, but for layers too wide
// for them).  The streaming
// kernels' time grows with the row tiles (each expands and multiplies on its own
// wave) and most where the activations no longer fit in LDS; the tiles keep fewer
// weights in flight per wave, so they gain least on weights that come from HBM.
// Streaming -> k groups, 7000 shapes of 1 ... 48 rows, graph-replayed over 340 MB of
// weights in turn (with eight in turn the same but for row-major weights, which
// come out 10-20 % better for the k groups from the caches):
//  - up to 16 rows, fragment-ordered weights: always streamed (16 x 6144 x 4096 5.5 ->
//    6.0 us, 8-bit 4-30 % slower: 12 x 4104 x 4096 6.6 -> 7.7).  Row-major ones:
//    mid-width layers of more k steps (257 ... 512 column groups 0.8-0.95 of the time);
//  - 17 to 32 rows, up to 256 groups: streamed (24 x 3584 x 6144 5.9 -> 7.2, 8-bit
//    24 x 3072 x 4096 6.6 -> 8.5; row-major 28 x 2048 x 6144 11.2 -> 12.6);
//  - 17 to 32, wider, fragment-ordered: k groups where the activations do not fit
//    (8-bit 30 x 7168 x 9216 31.7 -> 19.3), and for 4-bit codes at 257 ... 512 groups
//    (18 x 7168 x 3584 7.4 -> 6.0) and more k steps past 768 (20 x 16384 x 9216 18.6
//    -> 16.5; 20 x 12288 x 4096 8.4 -> 8.5); row-major from 16 steps (20 x 8192 x
//    4096 8.0 -> 6.8), wider 4-bit layers from 24;
//  - 33 to 48 rows: k groups (40 x 4608 x 9216 16.9 -> 10.9, 8-bit 48 x 5120 x 12288
//    39 -> 23), but for the shallowest K (up to 30 % slower), 8-bit codes past 512
//    groups while the activations fit (up to 15 % slower), and numbers of steps that
//    just fill passes of the streaming ring (13 ... 16; 25 ... 32 up to 36 rows: 33 x
//    2616 x 3776 5.0 -> 5.4) up to 256 groups;
//  - 33 to 48, past 1024 groups: while the activations fit, streamed (36 x 24576 x
//    2560 8-bit 14.6 -> 16.4), then not (44 x 37888 x 12288 146 -> 55); 4-bit codes
//    below 40 rows always.
// Where the k groups stand back K would be split across workgroups, whose scratch
// callers of so few rows do not provide.
constexpr int kFewRows = 48;
bool stream_weights(int M, int N, int K, int bits, bool frag) {
    if (M > kFewRows) return false;
    const int nk = (K * bits / 8 + kKB - 1) / kKB, groups = (N + 15) / 16, tm = (M + 15) / 16;
    const int cfg = choose_k_groups(M, N, K, bits).cfg;
    const bool fits = frag ? choose_frag_short(M, N, K, bits).whole : shared_lds_bytes(tm, nk) > 0;
    if (M > 32) {
        if (groups > 1024) return bits == 8 ? (frag ? fits : nk <= 4) : fits || M < 40;
        if (cfg < 0) return true;
        if (!frag) return nk <= (bits == 8 && groups > 512 ? 6 : 8);
        if (groups <= 256)
            return (bits == 8 && nk <= 6) || (nk > 12 && nk <= 16) || (bits == 4 && M <= 36 && nk > 24 && nk <= 32);
        return fits && (bits == 4 ? nk <= 8 : groups > 512 || nk <= 16);
    }
    if ((cfg != 10 && cfg != 11) || groups <= 256) return true;   // 64-row tiles would be half padding
    if (M > 16) {
        if (!frag) return nk < (bits == 4 && groups > 512 ? 24 : 16);
        return fits && (bits == 8 || (groups <= 512 ? nk <= 8 : groups <= 768 || nk <= 24));
    }
    if (frag) return true;
    return bits == 8 ? M <= 8 || nk < 30 || groups > 768 : M < 8 || nk <= 16 || groups > 512;
}

// Above 48 rows: whether k groups (plan p) beat the plan without them.  A k group
// takes w = nk / KG steps one after another, a workgroup of the K split `per` steps,
// and the split's second launch costs about 4 us; 8000 shapes of 49 ... 2000 rows,
// graph-replayed over 340 MB of weights in turn, other plan -> k groups:
//  - a shallow K leaves most groups idle: 128 x 128 x 64 3.0 -> 3.8 us, 200 x 8192 x
//    512 5.1 -> 6.1, 8-bit 160 x 1872 x 576 4.6 -> 5.1 (up to 64 rows of fragment-ordered
//    4-bit weights up to 12288 wide k groups are the faster ones there too);
//  - a deep K on few tiles: the split has more workgroups than CUs to share it, 64 x
//    64 x 65536 17 -> 29 us, 8-bit 250 x 64 x 65536 19 -> 61.  32 x 32 tiles hold up
//    to 8 steps a group, to 13 where the split is not two steps shorter or the
//    weights are read by several row tiles either way (64 x 2048 x 9216 8-bit 13.1 ->
//    16.6, 100 x 1024 x 9216 15.2 -> 11.0), and to 16 against long splits; 32 x 64
//    tiles to 16 steps (24 against six splits, 48 against four), 64 x 64 tiles
//    to 40 against four, to 64 at 8 bits;
//  - two groups are no faster than four waves of a 64 x 64 tile up to 16 steps at 8
//    bits and 28 at 4 bits (up to 25 % slower below; 5-15 % faster past it).
bool k_groups_faster(const Plan& p, const Plan& other, int M, int N, int nk, int bits, bool frag) {
    const bool shallow = !(frag && bits == 4 && M <= 64 && N <= 12288);
    const int w10 = (nk + 11) / 12, w11 = (nk + 7) / 8, w12 = (nk + 3) / 4;
    switch (p.cfg) {
        case 10:
            if (shallow && nk <= (bits == 8 ? 6 : 3)) return false;
            return w10 <= 8 || (w10 <= 13 && (M > 64 || other.per >= w10 - 1)) || (w10 <= 16 && other.per >= w10 - 2);
        case 11:
            if (shallow && nk <= (bits == 4 ? 6 : frag ? 9 : 7)) return false;
            return w11 <= (other.splits <= 4 ? 48 : other.splits <= 6 ? 24 : 16);
        case 12:
            if (shallow && nk <= (bits == 4 ? 7 : 9)) return false;
            return w12 <= (bits == 8 ? 64 : 40) || other.splits < 4;
        case 13: return other.cfg != 2 || nk >= (bits == 8 ? 20 : 32);
        default: return true;
    }
}

// The production plan (from measured sweeps on MI355X, graph-replayed with
// rotating weights):
//  - up to 48 rows where stream_weights says so: the short-M kernels (activations shared
//    in LDS for wide 4-bit layers, K split inside the workgroup otherwise);
//  - 4-bit codes with at least 448 tiles of 256 x 128 or of 128 x 128:
//    256 x 128 (eight waves of 64 x 64) at 448 ... 512 tiles of it, else
//    128 x 128 (four waves of 64 x 64) (see below);
//  - 8-bit codes (one MFMA per 64-byte k step, so operand reads from LDS weigh
//    twice as much per MFMA as for 4-bit codes): larger wave tiles.  128 x 256
//    (four waves of 64 x 128, two workgroups per CU; each wave reads 12
//    fragments per 32 MFMAs where 64 x 64 reads 8 per 16) from 512 of its
//    tiles; else 128 x 128 in two waves of 128 x 64 from 640 of its tiles
//    (three workgroups per CU fill the chip at 768); else 128 x 256 from 192
//    of its tiles; else 128 x 128 (four waves) from 192 of its tiles;
//  - at most 256 tiles of 32 x 32, 32 x 64, 64 x 64 or 64 x 128: the smallest
//    of these, in k groups (choose_k_groups);
//  - 129 ... 256 tiles of 128 x 128 and at least 128 k steps (48 for 8-bit codes,
//    49 up to 160 tiles): 128 x 128 with two k groups of four waves (see below);
//  - at least 512 tiles of 64 x 128: 64 x 128 (four waves of 64 x 32);
//  - otherwise 64 x 64 (four waves of 32 x 32); with few tiles (only where the
//    k groups stand back, see choose_k_groups) split over K across workgroups,
//    twice as deep for K >= 8192 and kept at 8 k steps or more per split.
Plan choose_plan(int M, int N, int K, int bits, bool k_groups, bool frag = false) {
    const bool few = k_groups ? stream_weights(M, N, K, bits, frag) : M <= kFewRows;
    const int nk = (K * bits / 8 + kKB - 1) / kKB;
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    if (!few && k_groups) {
        const Plan p = choose_k_groups(M, N, K, bits);
        if (p.cfg >= 0 && M <= kFewRows) return p;
        if (p.cfg >= 0 && k_groups_faster(p, choose_plan(M, N, K, bits, false), M, N, nk, bits, frag)) return p;
    }
    auto splits_for = [&](int t) {
        int s = t >= 256 ? 1 : (256 + t - 1) / t;
        if (K >= 8192 && t <= 256) s *= 2;
        const int cap = nk / 8 > 1 ? nk / 8 : 1;
        s = s < cap ? s : cap;
        return s < 32 ? s : 32;
    };
    Plan p;
    if (few) {
        // one wave per 16 columns, all M <= 48 tokens in its MFMA row tiles.  Wide
        // 4-bit layers whose activation codes fit in LDS share them among
        // ceil(groups / 256) waves per workgroup (one workgroup per CU); the rest
        // split K inside the workgroup, the more ways the fewer column groups
        // there are, keeping two batches per wave
        const int groups = (N + 15) / 16;
        const int tm = (M + 15) / 16;
        p = make_plan(M, N, K, 16 * tm, 16, 1, bits);
        if (bits == 4 && groups >= 768 && shared_lds_bytes(tm, nk) > 0) {
            p.cfg = 5;
            p.waves = (groups + 255) / 256 < kSharedMaxWaves ? (groups + 255) / 256 : kSharedMaxWaves;
        } else {
            const int u1 = tm == 1 ? 8 : 2, u4 = tm == 1 ? 4 : 2;
            int kw = groups >= 1024 ? 1 : groups >= 256 ? 2 : groups >= 128 ? 4 : 8;
            while (kw > 1 && (nk + (kw <= 2 ? u1 : u4) - 1) / (kw <= 2 ? u1 : u4) < 2 * kw) kw /= 2;
            p.cfg = 3;
            p.waves = kw;
        }
    } else if (tiles(128, 128) > 128 && tiles(128, 128) <= 256 &&
               nk >= (bits == 4 ? 128 : !k_groups ? 64 : tiles(128, 128) > 160 ? 48 : 49)) {
        // at most one 128 x 128 tile per CU and a deep K: two k groups of four
        // waves per tile (interleaved timings with rotating weights against the
        // plans below: 8-bit 1024 x 4096 x 4096 13 % faster, 1024 x 4096 x 12288
        // 15 %, 256 x 12288 x 4096 9 %, 1024 x 3584 x 18944 18 %; 4-bit
        // 1024 x 3584 x 18944 17 %, but 4 % slower at 1024 x 4096 x 12288 (96
        // k steps) and 6 % at 768 x 4096 x 12288, hence 128 k steps for 4-bit;
        // 8-bit at 56 k steps: 512 x 4608 x 3584 27.2 -> 23.1 us, 1000 x 3584 x
        // 3584 25.5 -> 22.3)
        p = make_plan(M, N, K, 128, 128, 1, bits);
        p.cfg = 9;
    } else if (bits == 4 && (tiles(256, 128) >= 448 || tiles(128, 128) >= 448)) {
        // 4-bit codes, from interleaved graph-replayed timings of both plans on
        // the layer-set shapes at 512 ... 16384 tokens: 256 x 128 wins only when
        // its 448 ... 512 tiles fill one round of two workgroups per CU (4096
        // tokens of the 3584- and 4096-wide layers, by 2-7 %); everywhere else
        // 128 x 128 (three workgroups per CU) is as fast or faster, by up to
        // 16 % where the 256 x 128 tiles leave a partly filled last round
        // (16384 x 4608: 6 % ; 4096 x 4608: 16 %) and 10 % over 64 x 128 at
        // 448 ... 511 tiles of 128 x 128
        const bool big = tiles(256, 128) >= 448 && tiles(256, 128) <= 512;
        p = make_plan(M, N, K, big ? 256 : 128, 128, 1, bits);
        p.cfg = big ? 0 : 1;
    } else if (bits == 8 && tiles(128, 256) >= 512) {
        // 8-bit codes, from timings with rotating weights of the LLaDA-shaped
        // layers at 128 ... 4096 tokens: 128 x 256 from 512 of its tiles 2-14 %
        // faster than 256 x 128 in eight waves; 768 tiles of 128 x 128 in two
        // waves (512 x 24576, 1024 x 12288) 12-15 % faster than four waves or
        // 128 x 256; 128 x 256 at 192 ... 511 of its tiles 9-16 % faster than
        // 128 x 128; below that 128 x 128 in four waves (1024 tokens of the
        // 4096-wide layers: 11-39 % faster than the larger tiles)
        p = make_plan(M, N, K, 128, 256, 1, bits);
        p.cfg = 7;
    } else if (bits == 8 && tiles(128, 128) >= 640) {
        p = make_plan(M, N, K, 128, 128, 1, bits);
        p.cfg = 8;
    } else if (bits == 8 && tiles(128, 256) >= 192) {
        p = make_plan(M, N, K, 128, 256, 1, bits);
        p.cfg = 7;
    } else if (bits == 8 && tiles(128, 128) >= 192) {
        p = make_plan(M, N, K, 128, 128, 1, bits);
        p.cfg = 1;
    } else if (tiles(128, 128) >= 512) {
        p = make_plan(M, N, K, 128, 128, 1, bits);
        p.cfg = 1;
    } else if (tiles(64, 128) >= 512) {
        p = make_plan(M, N, K, 64, 128, 1, bits);
        p.cfg = 4;
    } else {
        p = make_plan(M, N, K, 64, 64, splits_for(tiles(64, 64)), bits);
        p.cfg = 2;
    }
    return p;
}

// The plan of one call, weights row-major or in fragment order.
Plan gemm_plan(int M, int N, int K, int bits, bool frag) {
    if (frag && stream_weights(M, N, K, bits, true)) return choose_frag_short(M, N, K, bits);
    return choose_plan(M, N, K, bits, true, frag);
}

// What callers provide is what the K split across workgroups takes on every
// small grid, also where k groups run in its place and leave it unused: the size
// is part of the interface, so calls are accepted and refused by one rule.
size_t plan_workspace_bytes(int M, int N, int K, int bits) {
    const Plan p = choose_plan(M, N, K, bits, false);
    return p.splits > 1 ? (size_t)p.splits * M * N * 4 : 0;
}

}  // namespace
}  // namespace sq
