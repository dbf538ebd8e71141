// attn_fwd_kernel.h -- single-pass attention forward (Eq. 3) for gfx950, with the
// K and V tiles streamed into LDS by direct global->LDS copies.
//
// One workgroup covers 128 query rows of one (batch, head) (64 or 256 in the
// other geometries, see Geom).  Its waves are
// split in two halves over the key tiles (the first half of the tiles and the
// second; four quarters in one geometry), and at the end the parts of every
// row are merged through LDS.
// A wave owns QB blocks of 32 query rows: QB = 2 when D <= 64 (4 waves per
// 128-row workgroup), QB = 1 above (8 waves).  With QB = 2 every K and V^T operand
// read from LDS feeds two MFMAs.  Registers are budgeted for two waves per
// SIMD (256 each), or for one (up to 512) where the LDS already limits a CU
// to one wave per SIMD.
// Key/value tiles of 64 keys move through two to five LDS buffers per half:
// while one tile is consumed the next are copied straight from global memory
// (global_load_lds, 16 bytes per lane, no registers involved), keeping the
// row-major [key][d] layout.  Per 32-key sub-tile, wave and query block:
//
//   S^T = K Q^T      32x32x16 MFMA.  A = K rows read from LDS (16 bytes per
//                    lane), B = Q^T held in registers for the whole kernel.
//                    The accumulator puts one query per lane (lane % 32) and
//                    16 of the 32 keys in that lane, so the row maximum needs a
//                    single exchange between lane halves.
//   p = 2^(c (s-m))  c = |scale| log2(e), one multiply (or FMA) and one
//                    exponential per score.  m is fixed at the maximum of each
//                    wave's first sub-tile less kPBias / c, kPBias = 8 (p may then exceed 1); a row
//                    whose later logits would overflow the rounded p sends the
//                    workgroup through an exact fallback in which m moves, with
//                    the rescale of O and l, whenever a weight would pass 2^15.
//                    The bias keeps the largest weights near 2^8 instead of 1,
//                    so weights down to 2^-32 of the largest survive rounding
//                    to fp16 (its subnormals end at 2^-24): on very long key
//                    sequences their sum is otherwise lost.
//   O^T += V^T P^T   32x32x16 MFMA.  B = P straight from the S^T registers;
//                    A = V^T, produced from the row-major V tile by the
//                    transposing LDS read ds_read_b64_tr_b16: 16 lanes each
//                    point at 4 consecutive d of one key, and every lane gets
//                    4 consecutive keys of one d.
//   l                row sum of the rounded p.  When D is not a multiple of 32
//                    (and the LDS has room for it), the lanes whose d lies past
//                    D read a constant block instead of V: a one at d = D and
//                    zeros beyond, so the P V product also yields l in row D of
//                    O^T.  Otherwise the packed p pairs are summed with v_dot2
//                    against (1, 1).
//
// With the maximum fixed the pass is a software pipeline, so that each step's
// softmax has the independent MFMAs of its neighbours beside it: over the whole
// key range, in a written order, where the LDS holds the buffers for it
// (stream_tiles); else over one 64-key tile, left to the compiler's scheduler.
//
// This is the block-wise ("multi-stage") reduction of Sec. 3.2.1 -- a block's
// maximum and exponential sum merged into the running pair, and the key
// halves merged by the same rule -- fused with the element-wise normalisation
// and the product with V, so the N x M matrix A never leaves the chip (the
// IO-aware tiling of FlashAttention, Sec. 3.2.2).
//
// The kernel templates live in this header; attn_fwd.hip instantiates them
// for fp16 (and holds the entry points), attn_fwd_bf16.hip for bf16, so the
// two halves compile in parallel.
#pragma once

#include <utility>

#include "attn_geom.h"
#include "device.h"
#include "launch.h"

namespace sdattn {

namespace {

// The exponent's reference c m sits kPBias below the logit maximum it was
// taken from (weights of the largest logits near 2^8; see p = 2^(c (s - m))
// above); the online path moves m once a sub-tile's maximum would give a
// weight above 2^kRescaleLimit (fp16 holds values below 2^16).
constexpr float kPBias = 8.0f;
constexpr float kRescaleLimit = 15.0f;
constexpr int kDirectTiles = 4;         // tiles per key split up to which m moves from the start

template <int ET, int D, bool STATS, bool OROWS, int GEO>
__global__ __launch_bounds__((Geom<D, GEO>::kThreads), (Geom<D, GEO>::kWavesPerSimd)) void attn_fwd_lds_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ LS, int Lq, int Lk, float scale_abs, float c,
    float bias, int neg, int nqb, int oh) {
    using G = Geom<D, GEO>;
    static_assert(!G::kStream || G::QB == 2, "the streaming loop's step x works on query block x");
    constexpr int DK = G::DK;
    constexpr int DN = G::DN;
    constexpr int DD = G::DD;
    constexpr int QB = G::QB;
    constexpr int kQW = G::kQW;
    constexpr int kWaves = G::kWaves;
    constexpr int kThreads = G::kThreads;
    constexpr int TB = G::kTileBytes;

    extern __shared__ __attribute__((aligned(16))) char smem[];

    const int tid = threadIdx.x;
    const int lane = lane_id();
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kh = wave / kQW;         // key split ("half" when there are two) of this wave
    const int wq = wave % kQW;         // query slot of this wave

    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int bh = tile / nqb;
    const int qb = tile - bh * nqb;
    const int q0 = qb * G::kBQ + wq * 32 * QB;   // first row of this wave's QB blocks

    const char* Kh = (const char*)(K + (size_t)bh * Lk * D);
    const char* Vh = (const char*)(V + (size_t)bh * Lk * D);
    const int hbase = kh * G::kHalfBytes;   // this split's buffers
    const uint32_t lds0 = lds_offset(smem);

    // Tiles of this split: [t_first, t_first + t_count).  Split s takes
    // tiles s * nh .. s * nh + nh - 1 (nh = ceil(ntiles / kKS)), the last
    // ones what remains, possibly none; all run nh steps.
    constexpr int kTK = G::kTK;
    const int ntiles = (Lk + kTK - 1) / kTK;
    const int nh = (ntiles + G::kKS - 1) / G::kKS;
    const int t_first = kh * nh;
    const int t_count = min(nh, max(0, ntiles - t_first));

    // Copy tile t of this split into its buffer b (the split's kQW waves issue
    // the 1 KiB pieces wq, wq + kQW, ...).  What lies past the last key repeats
    // its last 16 bytes (finite data; their weights are forced to zero).
    auto issue_tile = [&](int t, int b) __attribute__((always_inline)) {
        // a tile is one contiguous run of K (and of V) rows; byte offsets inside a
        // head fit 32 bits (the launch checks Lk * D)
        const uint32_t dst = lds0 + hbase + b * G::kBufBytes;
        const uint32_t tile_off = (uint32_t)t * TB + lane * 16;
        const uint32_t last = (uint32_t)Lk * (2 * D) - 16;   // a head's last 16 bytes
#pragma unroll
        for (int i = 0; i < (2 * G::kChunks + kQW - 1) / kQW; ++i) {
            const int cidx = wq + kQW * i;
            if (cidx < 2 * G::kChunks) {
                const bool isv = cidx >= G::kChunks;
                const uint32_t off = tile_off + (isv ? cidx - G::kChunks : cidx) * 1024;
                copy16_to_lds(isv ? Vh : Kh, min(off, last), dst + cidx * 1024);
            }
        }
    };
    // Workgroup barrier with the copies of at most `ahead` (0 to 2) of this
    // wave's tiles still in flight.
    auto barrier = [&](int ahead) __attribute__((always_inline)) {
        constexpr int kMost = (2 * G::kChunks + kQW - 1) / kQW, kRem = 2 * G::kChunks % kQW;
        __builtin_amdgcn_sched_barrier(0);
        if (ahead <= 0) wait_copies<0>();
        else if (ahead == 1 && (kRem == 0 || wq < kRem)) wait_copies<kMost>();
        else if (ahead == 1) wait_copies<kMost - 1>();
        else if (kRem == 0 || wq < kRem) wait_copies<2 * kMost>();
        else wait_copies<2 * (kMost - 1)>();
        asm volatile("s_barrier" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    if constexpr (G::kStream) {
#pragma unroll
        for (int i = 0; i < G::kSlots - G::kStep; ++i)
            if (i < t_count) issue_tile(t_first + i, i);
    }

    // Constant block: a one in column 0 of every row, zeros elsewhere.  Lanes
    // whose d lies at or past D read it instead of V.
    if constexpr (G::kOnes) {
        const uint32_t one = from_float<ET>(1.0f);
        for (int i = tid; i < TB / 16; i += kThreads) {
            u32x4 w = {0u, 0u, 0u, 0u};
            if ((i * 8) % D == 0) w[0] = one;
            *(u32x4*)(smem + G::kConst + i * 16) = w;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }

    // Q^T operand of block j: lane holds query q0 + 32j + l32, d = 16s + 8*half .. +7.
    u32x4 qreg[QB][DK];
#pragma unroll
    for (int j = 0; j < QB; ++j)
#pragma unroll
        for (int s = 0; s < DK; ++s) {
            const int qrow = q0 + 32 * j + l32;
            const int d0 = 16 * s + 8 * half;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (qrow < Lq && d0 < D) v = *(const u32x4*)(Q + ((size_t)bh * Lq + qrow) * D + d0);
            if (neg) v ^= 0x80008000u;   // fold a negative scale into Q (exact)
            qreg[j][s] = v;
        }


    // Per-lane LDS byte offsets inside a buffer.
    // K rows: lane reads key row l32 at d = 8*half (+16 s, +32 sub rows).
    const int k_off = (l32 * D + 8 * half) * 2;
    // V^T via transposing reads: 16-lane group g = lane / 16 covers keys
    // 4*(g/2) .. +3 and d = 32n + 16*(g%2) .. +15; its lane i points at key
    // 4*(g/2) + i/4, d = 32n + 16*(g%2) + 4*(i%4) .. +3.
    int v_off[DN];
    int v_mask = -1;   // last d tile: 0 in the lanes that read the constant block
    int v_idx = 0;     // places of the sparse tile's values (see step32)
    {
        const int g = lane >> 4, i = lane & 15;
        const int krow = 4 * (g >> 1) + (i >> 2);
#pragma unroll
        for (int n = 0; n < DN; ++n) {
            int key = krow, ds = 32 * n + 16 * (g & 1) + 4 * (i & 3);
            if (G::kSparse && n == DD) {
                // the sparse tile: the lane's 16 lanes cover keys 16*(g/2) .. +15 and
                // d = 32n + 8*(g%2) .. +7; it points at key {0, 1, 8, 9}[i/4] (+ 2 when
                // i%4 >= 2) and 4 of those d.  The second read is 4 keys on.
                key = 16 * (g >> 1) + ((i >> 2) & 1) + 8 * (i >> 3) + 2 * ((i >> 1) & 1);
                ds = 32 * n + 8 * (g & 1) + 4 * (i & 1);
                v_idx = (i & 8) ? 0xeeee : 0x4444;
            }
            // past D: the constant block, or (without one) V columns 32
            // lower, whose finite products land in O^T rows never stored
            v_off[n] = ds < D ? TB + (key * D + ds) * 2
                              : G::kOnes ? G::kConst + (key * D + ds - D) * 2 : TB + (key * D + ds - 32) * 2;
            if (G::kOnes && ds >= D) v_mask = 0;
        }
    }
    // address of d tile n's values in the V tile of the buffer at LDS offset buf
    auto v_addr = [&](int buf, int n) __attribute__((always_inline)) -> const char* {
        return smem + ((G::kOnes && n == DN - 1 ? buf & v_mask : buf) + v_off[n]);
    };

    f32x16 acc[QB][DN];
    float m_run[QB];   // the exponent's reference m, in units of the raw scores
    float s_max[QB];   // true running max of the raw scores (this lane's keys)
    float l_part[QB];  // this lane's part of the row sum (v_dot2 path)
    auto reset = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < QB; ++j) {
#pragma unroll
            for (int n = 0; n < DN; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[j][n][r] = 0.0f;
            m_run[j] = -__builtin_inff();
            s_max[j] = -__builtin_inff();
            l_part[j] = 0.0f;
        }
    };
    reset();

    // p = 2^(c (s - m)).  How a sub-tile treats m (in raw score units; `bias` is
    // kPBias / c):
    //   kFirst  the wave's first sub-tile: m = its row maximum - bias (O is
    //           still 0)
    //   kFixed  m stays; p may exceed 1, and if a later logit exceeds the first
    //           sub-tile's maximum by more than ~8 (log2 units) the rounded p
    //           overflows to inf, which the overflow vote after the loop detects
    //   kOnline m moves (with the rescale of O and l) to a sub-tile's maximum
    //           - bias whenever that maximum would give a weight above
    //           2^kRescaleLimit -- the fallback
    enum { kFirst = 0, kFixed = 1, kOnline = 2 };

    // kOnline: move m (block j) for a row maximum mx, if any row of the wave has to.
    // m = -inf before the first keys (also where c = 0, when nothing else moves it).
    auto move_m = [&](int j, float mx) __attribute__((always_inline)) {
        if (__any(m_run[j] == -__builtin_inff() || (mx - m_run[j]) * c > kRescaleLimit)) {
            const float m_new = fmaxf(m_run[j], mx - bias);
            const float alpha = m_run[j] == -__builtin_inff() ? 0.0f : fast_exp2((m_run[j] - m_new) * c);
#pragma unroll
            for (int n = 0; n < DN; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[j][n][r] *= alpha;
            l_part[j] *= alpha;
            m_run[j] = m_new;
        }
    };

    // One 32-key sub-tile (keys kbase ..) held at row offset `sub` * 32 of
    // the tile in buffer base `buf`.
    auto step32 = [&](auto mode_c, auto tail_c, int buf, int sub, int kbase)
                      __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode_c)::value;
        constexpr bool TAIL = decltype(tail_c)::value;
        // ---- S^T = K Q^T, one K operand read for the QB blocks
        f32x16 st[QB];
#pragma unroll
        for (int j = 0; j < QB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) st[j][r] = 0.0f;
#pragma unroll
        for (int s = 0; s < DK; ++s) {
            u32x4 a = *(const u32x4*)(smem + buf + k_off + (32 * sub * D + 16 * s) * 2);
#pragma unroll
            for (int j = 0; j < QB; ++j) st[j] = mfma32x32x16<ET>(a, qreg[j][s], st[j]);
        }
        u32x4 pk[QB][2];
#pragma unroll
        for (int j = 0; j < QB; ++j) {
            if constexpr (TAIL) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kbase + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (key >= Lk) st[j][r] = -__builtin_inff();
                }
            }
            // ---- row maximum (Eq. 4's L), where the mode needs it
            if constexpr (MODE != kFixed || STATS) {
                float mloc = st[j][0];
#pragma unroll
                for (int r = 1; r < 16; ++r) mloc = fmaxf(mloc, st[j][r]);
                s_max[j] = fmaxf(s_max[j], mloc);
                if constexpr (MODE != kFixed) mloc = half_max(mloc);
                if constexpr (MODE == kFirst) m_run[j] = mloc - bias;
                else if constexpr (MODE == kOnline) move_m(j, mloc);
            }
            // ---- p = 2^(c (s - m)), rounded to the input type
            float p[16];
            const float negm = -m_run[j] * c;
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = fast_exp2(fmaf(st[j][r], c, negm));
            if constexpr (TAIL) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = kbase + 8 * (r >> 2) + 4 * half + (r & 3);
                    if (key >= Lk) p[r] = 0.0f;
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    pk[j][u][w] = pack2<ET>(p[8 * u + 2 * w], p[8 * u + 2 * w + 1]);
            if constexpr (!G::kOnes) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int w = 0; w < 4; ++w) l_part[j] = add_pair<ET>(pk[j][u][w], l_part[j]);
            }
        }
        // ---- O^T += V^T P^T; keys of operand slot e: 16u + 8*(e/4) + 4*half + e%4
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int n = 0; n < DD; ++n) {
                const char* vb = v_addr(buf, n) + (32 * sub + 16 * u) * D * 2;
                const u32x2 lo = lds_read_tr(vb);
                const u32x2 hi = lds_read_tr(vb + 8 * D * 2);
                const u32x4 a = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
                for (int j = 0; j < QB; ++j) acc[j][n] = mfma32x32x16<ET>(a, pk[j][u], acc[j][n]);
            }
        // The last 8 or 16 rows of V^T would fill a quarter or half of a dense
        // tile.  As a sparse tile each takes two rows, one with the first and one
        // with the last two of every four keys, and both 16-key steps take one
        // instruction.  Rows 0..7 and 8..15 of the tile are the two parts of d =
        // 32*DD .. +7, rows 16..23 and 24..31 those of the next 8 (or the row of ones).
        if constexpr (G::kSparse) {
            const char* vb = v_addr(buf, DD) + 32 * sub * D * 2;
            const u32x2 lo = lds_read_tr(vb);
            const u32x2 hi = lds_read_tr(vb + 4 * D * 2);
            const u32x4 a = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
            for (int j = 0; j < QB; ++j)
                acc[j][DD] = smfmac32x32x32<ET>(a, pk[j][0], pk[j][1], acc[j][DD], v_idx);
        }
    };

    // Add the two parts of the sparse tile's rows: registers 0..7 then hold d =
    // 32*DD .. +15 as in a dense tile.
    auto fold_sparse = [&]() __attribute__((always_inline)) {
        if constexpr (G::kSparse) {
#pragma unroll
            for (int j = 0; j < QB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[j][DD][r] += acc[j][DD][4 + r];
                    acc[j][DD][4 + r] = acc[j][DD][8 + r] + acc[j][DD][12 + r];
                }
        }
    };

    std::integral_constant<bool, false> full_c;
    std::integral_constant<bool, true> tail_c;
    std::integral_constant<int, kFirst> first_c;
    std::integral_constant<int, kFixed> fixed_c;
    std::integral_constant<int, kOnline> online_c;

    // A whole 64-key tile, written as a software
    // pipeline over the (sub-tile, block) pairs P0 = (0, 0), P1 = (0, 1), ...:
    //   S^T of sub-tile 0, then S^T of sub-tile 1 beside the softmax of P0,
    //   then the P V product of P(k-1) beside the softmax of Pk, and last
    //   the P V product of the last pair
    // so that each softmax has independent MFMAs next to it.  The compiler
    // schedules the whole tile: fences between these steps, or exponentials
    // pinned between the MFMAs, measured 1-2 % slower.
    //
    // In kOnline the tile's maximum (both sub-tiles, all rows at once) is taken
    // between the S^T products and the softmax, and m moves where it has to: one
    // look per tile, and the rest of the pipeline unchanged.
    auto tile_pipe = [&](auto mode_c, int buf) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode_c)::value;
        constexpr int NP = 2 * QB;               // (sub-tile, block) pairs
        f32x16 st[2][QB];
        u32x4 pk[2][QB][2];
        u32x4 vt[2][2][DD > 0 ? DD : 1];
        u32x4 vs[2];
        auto qk = [&](int sub) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < QB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) st[sub][j][r] = 0.0f;
#pragma unroll
            for (int s = 0; s < DK; ++s) {
                u32x4 a = *(const u32x4*)(smem + buf + k_off + (32 * sub * D + 16 * s) * 2);
#pragma unroll
                for (int j = 0; j < QB; ++j) st[sub][j] = mfma32x32x16<ET>(a, qreg[j][s], st[sub][j]);
            }
        };
        auto read_vt = [&](int sub) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int n = 0; n < DD; ++n) {
                    const char* vb = v_addr(buf, n) + (32 * sub + 16 * u) * D * 2;
                    const u32x2 lo = lds_read_tr(vb);
                    const u32x2 hi = lds_read_tr(vb + 8 * D * 2);
                    vt[sub][u][n] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                }
            if constexpr (G::kSparse) {
                const char* vb = v_addr(buf, DD) + 32 * sub * D * 2;
                const u32x2 lo = lds_read_tr(vb);
                const u32x2 hi = lds_read_tr(vb + 4 * D * 2);
                vs[sub] = u32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        };
        auto softmax = [&](int pr) __attribute__((always_inline)) {
            const int sub = pr / QB, j = pr % QB;
            float p[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = fast_exp2(fmaf(st[sub][j][r], c, -m_run[j] * c));
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    pk[sub][j][u][w] = pack2<ET>(p[8 * u + 2 * w], p[8 * u + 2 * w + 1]);
            if constexpr (!G::kOnes) {
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int w = 0; w < 4; ++w) l_part[j] = add_pair<ET>(pk[sub][j][u][w], l_part[j]);
            }
        };
        auto pv = [&](int pr) __attribute__((always_inline)) {
            const int sub = pr / QB, j = pr % QB;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int n = 0; n < DD; ++n) acc[j][n] = mfma32x32x16<ET>(vt[sub][u][n], pk[sub][j][u], acc[j][n]);
            if constexpr (G::kSparse)
                acc[j][DD] = smfmac32x32x32<ET>(vs[sub], pk[sub][j][0], pk[sub][j][1], acc[j][DD], v_idx);
        };
        qk(0);
        qk(1);
        if constexpr (MODE == kOnline || STATS) {
#pragma unroll
            for (int j = 0; j < QB; ++j) {
                float mx = fmaxf(st[0][j][0], st[1][j][0]), my = fmaxf(st[0][j][1], st[1][j][1]);
#pragma unroll
                for (int r = 2; r < 16; r += 2) {
                    mx = fmaxf(mx, fmaxf(st[0][j][r], st[1][j][r]));
                    my = fmaxf(my, fmaxf(st[0][j][r + 1], st[1][j][r + 1]));
                }
                mx = fmaxf(mx, my);
                s_max[j] = fmaxf(s_max[j], mx);
                if constexpr (MODE == kOnline) move_m(j, half_max(mx));
            }
        }
        read_vt(0);
        softmax(0);
#pragma unroll
        for (int k = 1; k < NP; ++k) {
            if (k == QB) read_vt(1);
            pv(k - 1);
            softmax(k);
        }
        if (QB == 1) read_vt(1);
        pv(NP - 1);
    };

    // consume the tile t (in buffer b) of this half; its first sub-tile in
    // mode mode0_c, the others in mode_c.
    auto consume = [&](auto mode0_c, auto mode_c, int t, int b) __attribute__((always_inline)) {
        const int buf = hbase + b * G::kBufBytes;
        const int kbase = t * kTK;
        // (kFirst is the pipeline's kOnline with nothing before it; the streaming
        // kernels' kFixed has its own loop)
        constexpr bool kPipelined = decltype(mode_c)::value == kOnline ||
                                    (!G::kStream && decltype(mode0_c)::value == kFixed);
        if (kbase + kTK <= Lk) {
            if constexpr (kPipelined) {
                tile_pipe(mode_c, buf);
            } else {
                step32(mode0_c, full_c, buf, 0, kbase);
                step32(mode_c, full_c, buf, 1, kbase + 32);
            }
        } else {
            if (kbase + 32 <= Lk) step32(mode0_c, full_c, buf, 0, kbase);
            else step32(mode0_c, tail_c, buf, 0, kbase);
            const int kb = kbase + 32;
            if (kb + 32 <= Lk) step32(mode_c, full_c, buf, 1, kb);
            else if (kb < Lk) step32(mode_c, tail_c, buf, 1, kb);
        }
    };

    // all tiles of this half: the first tile opens with kFirst, every other
    // sub-tile runs in mode_c (kFixed, or kOnline for the fallback)
    auto run_tiles = [&](auto mode_c) __attribute__((always_inline)) {
        if (t_count > 0) issue_tile(t_first, 0);
        barrier(0);
        if (t_count > 0) {
            if (t_count > 1) issue_tile(t_first + 1, 1);
            consume(first_c, mode_c, t_first, 0);
        }
        barrier(0);
        // Inside the loop only whole tiles are consumed; a ragged last tile
        // (the last tile of its half: nothing is copied over it afterwards)
        // waits in its buffer until the loop ends.  With a single way through
        // the loop body the accumulators keep their registers across
        // iterations instead of being copied at a join.
        int pend = -1;
        for (int i = 1; i < nh; ++i) {
            const int b = i & 1;
            if (i + 1 < t_count) issue_tile(t_first + i + 1, b ^ 1);
            if (i < t_count) {
                if ((t_first + i + 1) * kTK <= Lk) consume(mode_c, mode_c, t_first + i, b);
                else pend = i;
            }
            barrier(0);
        }
        if (pend >= 0) consume(mode_c, mode_c, t_first + pend, pend & 1);
    };

    // The fixed-maximum pass as one stream over the wave's (32-key sub-tile,
    // query block) pairs p = 0, 1, ...: step p issues
    //   S^T of pair p + 2,  p of pair p + 1,  O^T += of pair p
    // which do not depend on each other, a few exponentials behind each MFMA, in
    // the order written here (sched_barrier keeps it).  A wave issues in order,
    // so a run of MFMAs or of exponentials leaves the other unit idle; measured
    // on the bare mix of D = 40 (6 MFMAs, 16 multiplies, 16 exponentials, 8
    // conversions, two waves a SIMD), 198 clocks of MFMA and 233 of VALU take
    // 277 interleaved, 314 as two runs.  m enters as the initial value of S^T,
    // so that one multiply is left before the exponential.  Pair p's S^T and
    // rounded p live in the buffers of p's parity.  64x64 level (B2 H8 L4096 D40):
    // 56.6 -> 52.6 us; of a workgroup's 96.9 thousand clocks 88.4 are the loop's, 345 a
    // pair and SIMD for 6 MFMAs, 16 exponentials and 24 other operations (277 bare)
    // and the barriers, copies and LDS reads between them, at 1.9 to 2.0 GHz; in runs of
    // seconds the power limit takes the clock to about 1.65 GHz, and a launch 61 us.
    auto stream_tiles = [&]() __attribute__((always_inline)) {
        constexpr int SL = G::kSlots;
        constexpr int NQ = DK;                                 // MFMAs of S^T
        constexpr int NP = 2 * DD + (G::kSparse ? 1 : 0);      // MFMAs of O^T
        constexpr int NM = NQ + NP;
        const int n_whole = max(0, min(t_count, Lk / kTK - t_first));

        barrier(min(t_count, SL - G::kStep) - 1);   // tile 0 (the first SL - kStep were issued above)

        u32x4 kf[2][DK];
        u32x4 vf[2][2][DD > 0 ? DD : 1];
        u32x4 vsf[2];
        f32x16 st[2];
        u32x4 pk[2][2];
        f32x16 cin[QB];
        float negm[QB];   // -c m, with statistics

        auto read_k = [&](int buf, int sub, int s) __attribute__((always_inline)) {
            kf[sub][s] = *(const u32x4*)(smem + buf + k_off + (32 * sub * D + 16 * s) * 2);
        };
        // operand h of the O^T MFMAs (u = h / DD, n = h % DD; last the sparse one)
        auto read_v = [&](int buf, int sub, int h) __attribute__((always_inline)) {
            if (G::kSparse && h == 2 * DD) {
                const char* vb = v_addr(buf, DD) + 32 * sub * D * 2;
                const u32x2 lo = lds_read_tr(vb);
                const u32x2 hi = lds_read_tr(vb + 4 * D * 2);
                vsf[sub] = u32x4{lo[0], lo[1], hi[0], hi[1]};
            } else {
                const int u = h / DD, n = h % DD;
                const char* vb = v_addr(buf, n) + (32 * sub + 16 * u) * D * 2;
                const u32x2 lo = lds_read_tr(vb);
                const u32x2 hi = lds_read_tr(vb + 8 * D * 2);
                vf[sub][u][n] = u32x4{lo[0], lo[1], hi[0], hi[1]};
            }
        };
        // The softmax of st[x] as a list of 2-score units, each stage one unit
        // behind the one before: c s', 2^, rounding (and the row sum).  With
        // statistics S^T starts from zero, for the exact maximum, and -c m is added
        // to c s (taken as s - m and then times c, 4 operations for 2, the streaming
        // loop was the slower one at D = 32 and 48: 300 heads of 128 rows, 512 keys, D = 32 10.5 -> 11.0 us, 9.9 now).
        constexpr int kIn = STATS ? 3 : 2, kOut = G::kOnes ? 1 : 2;
        constexpr int kOps = 8 * (kIn + 2 + kOut);
        auto softmax_op = [&](int x, int i) __attribute__((always_inline)) {
            int at = 0;
#pragma unroll
            for (int t = 0; t < 10; ++t) {
                if (t < 8) {
                    if (STATS) {
                        if (i == at) s_max[x] = fmaxf(s_max[x], fmaxf(st[x][2 * t], st[x][2 * t + 1]));
                        if (i == at + 1) st[x][2 * t] = fmaf(st[x][2 * t], c, negm[x]);
                        if (i == at + 2) st[x][2 * t + 1] = fmaf(st[x][2 * t + 1], c, negm[x]);
                    } else {
                        if (i == at) st[x][2 * t] *= c;
                        if (i == at + 1) st[x][2 * t + 1] *= c;
                    }
                    at += kIn;
                }
                if (t >= 1 && t < 9) {
                    if (i == at) st[x][2 * t - 2] = fast_exp2(st[x][2 * t - 2]);
                    if (i == at + 1) st[x][2 * t - 1] = fast_exp2(st[x][2 * t - 1]);
                    at += 2;
                }
                if (t >= 2) {
                    const int w = t - 2;
                    if (i == at) pk[x][w / 4][w % 4] = pack2<ET>(st[x][2 * w], st[x][2 * w + 1]);
                    if (!G::kOnes && i == at + 1) l_part[x] = add_pair<ET>(pk[x][w / 4][w % 4], l_part[x]);
                    at += kOut;
                }
            }
        };
        auto max_of = [&](int x) __attribute__((always_inline)) {
            float m = st[x][0];
#pragma unroll
            for (int r = 1; r < 16; ++r) m = fmaxf(m, st[x][r]);
            return m;
        };
        auto s_mfma = [&](int x, int sub, int s) __attribute__((always_inline)) {
            st[x] = mfma32x32x16<ET>(kf[sub][s], qreg[x][s], s == 0 ? cin[x] : st[x]);
        };
        auto o_mfma = [&](int x, int sub, int h) __attribute__((always_inline)) {
            if (G::kSparse && h == 2 * DD)
                acc[x][DN - 1] = smfmac32x32x32<ET>(vsf[sub], pk[x][0], pk[x][1], acc[x][DN - 1], v_idx);
            else
                acc[x][h % DD] = mfma32x32x16<ET>(vf[sub][h / DD][h % DD], pk[x][h / DD], acc[x][h % DD]);
        };
        // Step of parity X on sub-tile s (its place SUB in the tile).  Step 0 reads the
        // K of sub-tile s + 2 (kbuf), step 1 the V of s + 1 (vbuf): a whole sub-tile
        // ahead of the MFMAs they feed.
        auto step = [&](auto x_c, auto sub_c, int kbuf, int vbuf) __attribute__((always_inline)) {
            constexpr int X = decltype(x_c)::value, SUB = decltype(sub_c)::value;
#pragma unroll
            for (int g = 0; g < NM; ++g) {
                // S^T and O^T in turn; each is a chain on one accumulator, which two
                // instructions in a row would wait on
                const int q = (g * NQ + NM - 1) / NM, h = g - q;   // S^T and O^T MFMAs before this one
                if ((g + 1) * NQ > q * NM) s_mfma(X, SUB ^ 1, q);
                else o_mfma(X, SUB, !G::kSparse || h < DD ? h : h == DD ? 2 * DD : h - 1);
                __builtin_amdgcn_sched_barrier(0);
                if (X == 0 && g < NQ) read_k(kbuf, SUB, g);
                if (X == 1) {
#pragma unroll
                    for (int i = g * NP / NM; i < (g + 1) * NP / NM; ++i) read_v(vbuf, SUB ^ 1, i);
                }
#pragma unroll
                for (int i = g * kOps / NM; i < (g + 1) * kOps / NM; ++i) softmax_op(1 - X, i);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        std::integral_constant<int, 0> x0;
        std::integral_constant<int, 1> x1;

        if (n_whole > 0) {
            // pairs 0 and 1: their scores from zero, m from the first sub-tile's
            // maximum, then the rounded p of pair 0
            const int buf = hbase;
#pragma unroll
            for (int j = 0; j < QB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) cin[j][r] = 0.0f;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                if (x == 0) {
#pragma unroll
                    for (int s = 0; s < DK; ++s) read_k(buf, 0, s);
                }
#pragma unroll
                for (int s = 0; s < DK; ++s) s_mfma(x, 0, s);
            }
#pragma unroll
            for (int j = 0; j < QB; ++j) {
                m_run[j] = half_max(max_of(j)) - bias;
                negm[j] = -m_run[j] * c;
            }
#pragma unroll
            for (int x = 0; x < 2; ++x) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (!STATS) {
                        st[x][r] -= m_run[x];
                        cin[x][r] = -m_run[x];
                    }
            }
            if (STATS) s_max[0] = max_of(0);
#pragma unroll
            for (int r = 0; r < 16; ++r) st[0][r] = fast_exp2(STATS ? fmaf(st[0][r], c, negm[0]) : st[0][r] * c);
#pragma unroll
            for (int w = 0; w < 8; ++w) {
                pk[0][w / 4][w % 4] = pack2<ET>(st[0][2 * w], st[0][2 * w + 1]);
                if (!G::kOnes) l_part[0] = add_pair<ET>(pk[0][w / 4][w % 4], l_part[0]);
            }
#pragma unroll
            for (int s = 0; s < DK; ++s) read_k(buf, 1, s);
#pragma unroll
            for (int h = 0; h < NP; ++h) read_v(buf, 0, h);
        }
        int slot = 0;
        float s_last = 0.0f, l_last = 0.0f;
        for (int i = 0; i < nh; i += G::kStep) {
            // Tiles up to i + kStep are in LDS for every wave, and the buffers of the
            // tiles before i are free for the next kStep copies.
            barrier(min(t_count - 1, i + SL - 1 - G::kStep) - (i + G::kStep));
#pragma unroll
            for (int k = 0; k < G::kStep; ++k) {
                const int t = i + SL - G::kStep + k;
                const int b = slot - G::kStep + k;
                if (t < t_count) issue_tile(t_first + t, b < 0 ? b + SL : b);
            }
#pragma unroll
            for (int k = 0; k < G::kStep; ++k) {
                const int cur = hbase + slot * G::kBufBytes;
                slot = slot + 1 == SL ? 0 : slot + 1;
                const int nxt = hbase + slot * G::kBufBytes;
                if (i + k < n_whole) {
                    __builtin_amdgcn_sched_barrier(0);
                    step(x0, x0, nxt, 0);
                    step(x1, x0, 0, cur);
                    step(x0, x1, nxt, 0);
                    // the last step of a tile takes the softmax of the next tile's first
                    // pair: what it adds is dropped below if there is none
                    s_last = s_max[0];
                    l_last = l_part[0];
                    step(x1, x1, 0, nxt);
                }
            }
        }
        if (n_whole > 0) {
            s_max[0] = s_last;
            l_part[0] = l_last;
        }
        // a ragged last tile is the one after the whole ones; its copy has been
        // waited for by the barrier of the step before.  (consume's way for a whole
        // tile is never taken from here; without it the compiler spills 24 to 69 of
        // the loop's registers: 300 keys D = 40 7.2 -> 8.3 us)
        if (n_whole < t_count) {
            const int t = t_first + n_whole, b = n_whole % SL;
            if (n_whole > 0) consume(fixed_c, fixed_c, t, b);
            else consume(first_c, fixed_c, t, b);
        }
    };

    // With few tiles and one query block a moving m costs little beside the fixed
    // part, and rows with large logits need no second pass.  Fixed / moving, us, and with
    // queries four times as long: 16 heads of 256 rows and keys D = 160 8.0 / 7.9, 11.8 /
    // 8.0; 1024 rows, 512 keys D = 80 7.9 / 8.0, 11.6 / 8.0; 2048 rows, 512 keys D = 128
    // 27.0 / 26.9, 46.2 / 26.9; 300 rows and keys (a ragged tile) D = 80 6.6 / 7.1, 11.0 /
    // 7.4, the most that it costs (two query blocks: D = 64, 1024 keys 12.2 / 13.8, so not
    // for them).  At large D a ragged tile's steps are code of their own to fetch (Lk
    // 300, D = 160: 10.7 -> 11.9), so whole tiles only.  bf16 weights do not overflow.
    const bool direct = !G::kStream && QB == 1 && ET == kF16 && nh <= kDirectTiles &&
                        (DN <= 3 || Lk % kTK == 0);
    // Overflow vote: with m fixed at the first sub-tile's maximum - bias, a
    // later logit larger than that maximum by more than ~8 (log2) overflows
    // the rounded p to inf,
    // which makes this lane's row sum non-finite.  Any such row sends the
    // whole workgroup (it shares the LDS tiles) through the online path.
    int redo = 1;   // (one copy of the online path's code)
    if (!direct) {
        if constexpr (G::kStream) stream_tiles();
        else run_tiles(fixed_c);
        fold_sparse();
        bool overflow = false;
#pragma unroll
        for (int j = 0; j < QB; ++j) {
            float l_check;
            if constexpr (G::kOnes) {
                constexpr int dd = D % 32;
                constexpr int rsel = 4 * (dd >> 3) + (dd & 3);
                l_check = acc[j][D / 32][rsel];
            } else {
                l_check = l_part[j];
            }
            overflow = overflow || (__float_as_uint(l_check) & 0x7f800000u) == 0x7f800000u;   // inf or NaN
        }
        // workgroup-wide OR through LDS
        int* vote = (int*)(smem + G::kVote);
        const int wave_overflow = __any(overflow) ? 1 : 0;   // ballot with every lane active
        if (lane == 0) vote[wave] = wave_overflow;
        __syncthreads();
        redo = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) redo |= vote[w];
        __syncthreads();
    }
    if (redo) {
        reset();
        run_tiles(online_c);
        fold_sparse();
        // The merge below writes into the tile buffers; a wave of key
        // half 1 may still be reading its ragged last tile there (run_tiles
        // ends without a barrier after that tile).  The fixed-maximum pass
        // has the vote's barriers in between.
        __syncthreads();
    }

    if constexpr (STATS) {
#pragma unroll
        for (int j = 0; j < QB; ++j) s_max[j] = half_max(s_max[j]);
    }

    // ---- merge the key splits of every row (the block-merge rule): split s
    // > 0 leaves its O^T, m, max and l in LDS, split 0 folds them in.  Its latency
    // is all of a workgroup's last half microsecond, so: no branch for an empty
    // split, all splits unrolled, 16 bytes a lane (four splits, 16 heads, 512 keys:
    // D = 40 7.0 -> 6.2 us, D = 64 9.3 -> 8.5)
    constexpr int kMF = G::kRegs * 64 + 3 * 64;   // floats per query block
    auto mrg_of = [&](int s) { return (float*)smem + ((s - 1) * kQW + wq) * G::kMergeFloats; };
    if (kh != 0) {
        float* mrg = mrg_of(kh);
#pragma unroll
        for (int j = 0; j < QB; ++j) {
            float* mj = mrg + j * kMF;
#pragma unroll
            for (int i = 0; i < G::kRegs; i += 4)
                *(f32x4*)(mj + i * 64 + lane * 4) = f32x4{acc[j][i / 16][i % 16], acc[j][i / 16][i % 16 + 1],
                                                          acc[j][i / 16][i % 16 + 2], acc[j][i / 16][i % 16 + 3]};
            mj[G::kRegs * 64 + lane] = m_run[j];
            mj[G::kRegs * 64 + 64 + lane] = s_max[j];
            mj[G::kRegs * 64 + 128 + lane] = l_part[j];
        }
    }
    __syncthreads();
    if (kh != 0) return;
#pragma unroll
    for (int s = 1; s < G::kKS; ++s)
#pragma unroll
    for (int j = 0; j < QB; ++j) {
        const float* mj = mrg_of(s) + j * kMF;
        const float m_b = mj[G::kRegs * 64 + lane];
        const float m_new = fmaxf(m_run[j], m_b);
        // an empty split (m = -inf, O and l zero) may have any finite weight: finite
        // differences keep it so where c = 0
        const float a0 = fast_exp2(fmaxf(m_run[j] - m_new, -__FLT_MAX__) * c);
        const float a1 = fast_exp2(fmaxf(m_b - m_new, -__FLT_MAX__) * c);
#pragma unroll
        for (int i = 0; i < G::kRegs; i += 4) {
            const f32x4 w = *(const f32x4*)(mj + i * 64 + lane * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[j][i / 16][i % 16 + e] = acc[j][i / 16][i % 16 + e] * a0 + w[e] * a1;
        }
        s_max[j] = fmaxf(s_max[j], mj[G::kRegs * 64 + 64 + lane]);
        l_part[j] = l_part[j] * a0 + mj[G::kRegs * 64 + 128 + lane] * a1;
        m_run[j] = m_new;
    }

    // ---- epilogue: l, O / l, store
#pragma unroll
    for (int j = 0; j < QB; ++j) {
        float l;
        if constexpr (G::kOnes) {
            constexpr int dd = D % 32;               // position of the ones row in its d tile
            constexpr int hsel = (dd >> 2) & 1, rsel = 4 * (dd >> 3) + (dd & 3);
            const float own = acc[j][D / 32][rsel];
            const float other = half_partner(own, half);
            l = (half == hsel) ? own : other;
        } else {
            l = half_sum(l_part[j]);
        }
        const float inv = 1.0f / l;
        const int qrow = q0 + 32 * j + l32;
        if (qrow < Lq) {
            uint16_t* orow = OROWS ? out_base(O, bh, Lq, D, oh) + (size_t)qrow * out_stride(D, oh)
                                   : O + ((size_t)bh * Lq + qrow) * D;
#pragma unroll
            for (int n = 0; n < DN; ++n)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int d0 = 32 * n + 8 * g + 4 * half;
                    if (32 * n + 8 * g < D) {   // D % 8 == 0: then d0 + 3 < D for both halves
                        u32x2 w;
                        w[0] = pack2<ET>(acc[j][n][4 * g + 0] * inv, acc[j][n][4 * g + 1] * inv);
                        w[1] = pack2<ET>(acc[j][n][4 * g + 2] * inv, acc[j][n][4 * g + 3] * inv);
                        *(u32x2*)(orow + d0) = w;
                    }
                }
            if (LS && half == 0) {
                // Eq. 4 in natural units: L = max_j scale q.k, S = sum_j exp(scale q.k - L)
                float* o2 = LS + ((size_t)bh * Lq + qrow) * 2;
                o2[0] = s_max[j] * scale_abs;
                o2[1] = l * fast_exp2(fmaf(-s_max[j], c, m_run[j] * c));   // the weights' c m, rounded as theirs
            }
        }
    }
}

template <int ET, int D, bool STATS, bool OROWS, int GEO>
hipError_t launch_kernel(const AttnArgs& a) {
    using G = Geom<D, GEO>;
    const int nqb = (a.Lq + G::kBQ - 1) / G::kBQ;
    const long long nblk = (long long)a.B * a.H * nqb;
    const float scale_abs = a.scale < 0 ? -a.scale : a.scale;
    const float c = scale_abs * kLog2e;
    const float bias = c > 1e-30f ? kPBias / c : 0.0f;   // scale 0: every weight is 1 whatever m
    auto kern = attn_fwd_lds_kernel<ET, D, STATS, OROWS, GEO>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                                       G::kLdsBytes);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(G::kThreads), G::kLdsBytes,
                       (hipStream_t)a.stream, (const uint16_t*)a.q, (const uint16_t*)a.k,
                       (const uint16_t*)a.v, (uint16_t*)a.out, a.ls, a.Lq, a.Lk, scale_abs, c, bias,
                       a.scale < 0 ? 1 : 0, nqb, a.o_rows ? a.H : 0);
    return hipGetLastError();
}

template <int ET, int D, bool STATS, bool OROWS>
hipError_t launch_geo(const AttnArgs& a) {
    switch (pick_geometry<D>((long long)a.B * a.H, a.Lq, a.Lk)) {
        case kGeoSmall: return launch_kernel<ET, D, STATS, OROWS, kGeoSmall>(a);
        case kGeoQuarter:
            if constexpr (Geom<D, kGeoQuarter>::kFits) return launch_kernel<ET, D, STATS, OROWS, kGeoQuarter>(a);
            break;
        case kGeoBig:
            if constexpr (Geom<D, kGeoBig>::kFits) return launch_kernel<ET, D, STATS, OROWS, kGeoBig>(a);
            break;
        case kGeoPair:
            if constexpr (Geom<D, kGeoPair>::kFits) return launch_kernel<ET, D, STATS, OROWS, kGeoPair>(a);
            break;
        default: break;
    }
    return launch_kernel<ET, D, STATS, OROWS, kGeoNormal>(a);
}

// Statistics and merged heads are instantiated apart (attn_fwd_stats.hip has
// the former), so that the files compile side by side.
enum { kPlain = 0, kStats = 1 };

template <int ET, int D, int PART>
hipError_t launch_d(const AttnArgs& a) {
    if constexpr (!Geom<D, kGeoNormal>::kFits || !Geom<D, kGeoSmall>::kFits) {
        return launch_attn_fwd_generic(a);
    } else {
        if (a.ls && a.o_rows) return hipErrorInvalidValue;   // no caller asks for both
        // tile copies address a head's K and V with 32-bit byte offsets
        if ((long long)a.Lk * D * 2 > 0x7fffffffLL) return launch_attn_fwd_generic(a);
        if constexpr (PART == kStats) return launch_geo<ET, D, true, false>(a);
        else return a.o_rows ? launch_geo<ET, D, false, true>(a) : launch_geo<ET, D, false, false>(a);
    }
}

template <int ET, int PART, int... Ds>
hipError_t dispatch_d(const AttnArgs& a, std::integer_sequence<int, Ds...>) {
    hipError_t r = hipErrorInvalidValue;
    bool hit = ((a.D == 8 * (Ds + 1) ? (r = launch_d<ET, 8 * (Ds + 1), PART>(a), true) : false) || ...);
    return hit ? r : hipErrorInvalidValue;
}

}  // namespace

}  // namespace sdattn
