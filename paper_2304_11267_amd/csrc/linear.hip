// linear.hip -- the projections around the attention in SD's transformer
// blocks: y = x w^T + bias with weights stored [out, in], and the head
// split / merge folded into the addressing of the rows.
//
// A token row m = b*L + l of x (or y) lives either in rows layout [B, L, C]
// or in heads layout [B, H, L, C/H] (channel c = h*(C/H) + d at
// ((b*H + h)*L + l)*(C/H) + d).  Writing Q, K and V in heads layout is the
// head split before Eq. 3; reading O in heads layout is the head merge before
// the output projection -- neither needs a transpose of its own.
//
// Two kernels: linear_kernel shares 128x64 tiles among a workgroup's waves
// (below); linear_ksplit_kernel, for few tiles or few token rows, splits the
// reduced dimension over them (launch_group_e has the rule).
//
// One launch may carry up to three independent products (the block's Q, K
// and V projections, whose inputs differ for cross-attention), each possibly
// a batch of equal-sized products at fixed strides (the 36 products of a
// Winograd convolution); each workgroup finds its product and batch item
// from its tile index, so the small context projections run beside the
// large latent one instead of after it.
//
// Workgroup tile: 128 token rows x 64 output channels, four waves of 32 rows.
// Each 64-channel slice of the x and w tiles is copied global -> LDS with
// global_load_lds (16 bytes per lane, whole 128-byte rows per instruction,
// no registers), into a ring of kStages slices so that kStages - 1 copies are
// in flight while one slice is multiplied.  Inside a slice, row r's 16-byte
// chunk c sits at chunk position c ^ swz(r), which keeps the MFMA operand
// reads (ds_read_b128, one row per lane) free of bank conflicts.  The product
// runs as y^T = w x^T on 32x32x16 MFMAs: A = 32 weight rows x 16 channels,
// B = 16 channels x 32 token rows, one token row per lane; each lane ends with
// 4 consecutive output channels per register group; the tile goes out through
// LDS so that each lane stores 16 contiguous bytes.
#include "device.h"
#include "launch.h"

namespace sdattn {

namespace {

constexpr int kBM = 128;                          // token rows per workgroup
constexpr int kBN = 64;                           // output channels per workgroup
constexpr int kBK = 64;                           // input channels per slice
constexpr int kUnits = (kBM + kBN) * kBK / 8;     // 16-byte chunks per slice (1536)
constexpr int kSliceBytes = kUnits * 16;          // 24 KiB
constexpr int kCopies = kUnits / 64 / 4;          // copy instructions per wave per slice (6)
constexpr int kStages = 3;
constexpr int kRuns = 4;                          // partial sums over the input channels
constexpr int kSplitMinK = 512;                   // fewest channels (exclusive) summed that way
constexpr int kLdsBytes = kStages * kSliceBytes;  // 72 KiB: two workgroups per CU

struct LinProblem {
    const uint16_t* x;
    const uint16_t* w;
    const uint16_t* bias;   // null: no bias
    uint16_t* y;
    int M, K, N, L;         // M = B*L token rows
    int xhw, yhw;           // head widths of the heads layouts (1 for rows layout)
    int nnt, tile0;         // channel tiles; first tile index of this product
    int per_batch;          // tiles of one batch item
    long long sx, sw, sy;   // element strides between batch items
};
struct LinGroup {
    LinProblem p[kMaxLinearProblems];
    int n;
};

// chunk-position swizzle of row r: distinct for any 8 consecutive rows, and
// (r & 1, swz) distinct for any 16 consecutive rows
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// c / hw for 0 <= c < 2^16 and 8 <= hw: the fp32 quotient is within one of
// the true one, and one correction step makes it exact.
__device__ __forceinline__ int div_small(int c, int hw, float inv_hw) {
    int h = (int)((float)c * inv_hw);
    h -= (h * hw > c) ? 1 : 0;
    h += ((h + 1) * hw <= c) ? 1 : 0;
    return h;
}

// Element offset of token row m = b*L + l (channel 0, head 0) in a tensor of
// C channels, and of channel c relative to it.
template <bool HEADS>
__device__ __forceinline__ size_t row_base(int m, int L, int C, int hw) {
    if constexpr (HEADS) {
        const int b = m / L, l = m - b * L;
        return ((size_t)b * (C / hw) * L + l) * hw;
    } else {
        return (size_t)m * C;
    }
}
template <bool HEADS>
__device__ __forceinline__ size_t chan_offset(int c, int L, int hw, float inv_hw) {
    if constexpr (HEADS) {
        const int h = div_small(c, hw, inv_hw);
        return (size_t)h * L * hw + (c - h * hw);
    } else {
        return (size_t)c;
    }
}

// Wait until at most `ahead` slices of this wave's copies are still in flight.
__device__ __forceinline__ void wait_slices(int ahead) {
    static_assert(kStages == 3, "wait_slices covers ahead = 0 and 1");
    if (ahead >= 1) __builtin_amdgcn_s_waitcnt(vm_wait(kCopies));
    else __builtin_amdgcn_s_waitcnt(vm_wait(0));
}

// Workgroup barrier after this wave's LDS reads have returned.  The slice
// copies are waited for explicitly (wait_slices); a fence here would drain
// every copy still in flight, since they count as LDS writes.  The memory
// clobber keeps the compiler from moving LDS reads across the barrier.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int ET, bool XH, bool YH, bool FOLD>
__global__ __launch_bounds__(256) void linear_kernel(const LinGroup grp) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int pi = (grp.n > 2 && tile >= grp.p[2].tile0) ? 2 : (grp.n > 1 && tile >= grp.p[1].tile0) ? 1 : 0;
    const LinProblem& P = grp.p[pi];
    const int bi = (tile - P.tile0) / P.per_batch;     // batch item
    const int local = tile - P.tile0 - bi * P.per_batch;
    const uint16_t* __restrict__ X = P.x + bi * P.sx;
    const uint16_t* __restrict__ W = P.w + bi * P.sw;
    const int M = P.M, K = P.K, N = P.N, L = P.L, xhw = P.xhw;
    const int nt = local % P.nnt;        // consecutive workgroups share the token rows
    const int m0 = (local / P.nnt) * kBM;
    const int n0 = nt * kBN;
    const int nk = (K + kBK - 1) / kBK;

    // Copy j of this wave moves 16-byte chunk c of tile row r (x rows first,
    // then w rows); rows past M or N repeat the last row (their outputs are
    // never stored), channels past K repeat the last chunk (their operands are
    // zeroed before use).  Row bases are fixed across slices.
    size_t cbase[kCopies];
    int cch[kCopies];
#pragma unroll
    for (int j = 0; j < kCopies; ++j) {
        const int u0 = (wave * kCopies + j) * 64;
        const int u = u0 + lane;
        if (u0 < kBM * 8) {
            const int r = u >> 3;
            cch[j] = 8 * ((u & 7) ^ swz(r));
            cbase[j] = row_base<XH>(min(m0 + r, M - 1), L, K, xhw);
        } else {
            const int r = (u >> 3) - kBM;
            cch[j] = 8 * ((u & 7) ^ swz(r));
            cbase[j] = (size_t)min(n0 + r, N - 1) * K;
        }
    }
    const float inv_xhw = 1.0f / (float)xhw;

    // slice i (channels 64i .. 64i + 63) into ring slot i % kStages
    auto issue = [&](int i) __attribute__((always_inline)) {
        const int k0 = i * kBK;
        char* st = smem + (i % kStages) * kSliceBytes;
#pragma unroll
        for (int j = 0; j < kCopies; ++j) {
            const int u0 = (wave * kCopies + j) * 64;
            const int ch = min(k0 + cch[j], K - 8);
            const char* src = u0 < kBM * 8
                                  ? (const char*)(X + cbase[j] + chan_offset<XH>(ch, L, xhw, inv_xhw))
                                  : (const char*)(W + cbase[j] + ch);
            __builtin_amdgcn_global_load_lds(src, (lds_void_t*)(st + u0 * 16), 16, 0, 0);
        }
    };

    // operand offsets inside a slice: B = x row 32*wave + l32, A_t = w row
    // 32t + l32, chunk 2s + half for k-step s (rows 32t + l32 share swz(l32))
    const int hx = swz(l32);
    int offx[4], offw[2][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int cpos = (2 * s + half) ^ hx;
        offx[s] = ((32 * wave + l32) * 8 + cpos) * 16;
#pragma unroll
        for (int t = 0; t < 2; ++t) offw[t][s] = ((kBM + 32 * t + l32) * 8 + cpos) * 16;
    }

    // bias of this lane's output channels (8-byte aligned groups of 4),
    // fetched before the product
    const uint16_t* __restrict__ Bias = P.bias;
    u32x2 bias[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) bias[t][g] = u32x2{0u, 0u};
    if (Bias) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = min(n0 + 32 * t + 8 * g + 4 * half, N - 4);
                bias[t][g] = *(const u32x2*)(Bias + n);
            }
    }

    // acc += slice i (FIRST: acc = slice i); before() is issued while the slice's
    // operands come from LDS
    f32x16 zero;
#pragma unroll
    for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
    auto slice = [&](int i, auto first_c, f32x16 (&acc)[2], auto before) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_c)::value;
        wait_slices(min(nk - 1 - i, kStages - 2));
        lds_barrier();   // slice i is in LDS for every wave; slot (i - 1) % kStages is free
        if (i + kStages - 1 < nk) issue(i + kStages - 1);
        const char* st = smem + (i % kStages) * kSliceBytes;
        const int kval = K - i * kBK;    // channels of this slice inside K (uniform)
        // all twelve operand reads first, so their latencies overlap
        u32x4 bf[4], af[2][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            bf[s] = *(const u32x4*)(st + offx[s]);
            af[0][s] = *(const u32x4*)(st + offw[0][s]);
            af[1][s] = *(const u32x4*)(st + offw[1][s]);
        }
        before();
        if (kval < kBK) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (8 * (2 * s + half) >= kval) {
                    bf[s] = u32x4{0u, 0u, 0u, 0u};
                    af[0][s] = bf[s];
                    af[1][s] = bf[s];
                }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            acc[0] = mfma32x32x16<ET>(af[0][s], bf[s], FIRST && s == 0 ? zero : acc[0]);
            acc[1] = mfma32x32x16<ET>(af[1][s], bf[s], FIRST && s == 0 ? zero : acc[1]);
        }
    };

#pragma unroll
    for (int i = 0; i < kStages - 1; ++i)
        if (i < nk) issue(i);

    // With FOLD, acc sums a run of slices and tot the runs before it.  Past
    // kSplitMinK channels that is the split-K kernel's order of summation, so a
    // row has the same bits whichever kernel takes it, alone or in a batch of any
    // size; up to there the split kernel is not taken and one run does (the 64x64
    // level's convolution 27 us against 28).  The additions cost a wave that has its
    // SIMD to itself 5 clocks each, beside MFMAs too: without / with them 2048x640x640
    // 7.2 / 7.5 us (7.9 with them in the loop of every slice), 1024x1280x1280 11.3 /
    // 11.4 (12.0), 2048x2560x640 19.4 / 19.0 (20.0).
    f32x16 acc[2] = {zero, zero}, tot[2] = {zero, zero};
    const int run = K > kSplitMinK ? (nk + kRuns - 1) / kRuns : nk;
    if constexpr (!FOLD) {
        // (a loop of its own: as slices opened by a run's first one, products with a
        // ragged last slice were slower, 8192x328x320 8.7 -> 9.1 us)
        for (int i = 0; i < nk; ++i) {
            wait_slices(min(nk - 1 - i, kStages - 2));
            lds_barrier();   // slice i is in LDS for every wave; slot (i - 1) % kStages is free
            if (i + kStages - 1 < nk) issue(i + kStages - 1);
            const char* st = smem + (i % kStages) * kSliceBytes;
            const int kval = K - i * kBK;    // channels of this slice inside K (uniform)
            // all twelve operand reads first, so their latencies overlap
            u32x4 bf[4], af[2][4];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                bf[s] = *(const u32x4*)(st + offx[s]);
                af[0][s] = *(const u32x4*)(st + offw[0][s]);
                af[1][s] = *(const u32x4*)(st + offw[1][s]);
            }
            if (kval < kBK) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    if (8 * (2 * s + half) >= kval) {
                        bf[s] = u32x4{0u, 0u, 0u, 0u};
                        af[0][s] = bf[s];
                        af[1][s] = bf[s];
                    }
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                acc[0] = mfma32x32x16<ET>(af[0][s], bf[s], acc[0]);
                acc[1] = mfma32x32x16<ET>(af[1][s], bf[s], acc[1]);
            }
        }
    } else
    for (int i0 = 0; i0 < nk; i0 += run) {
        slice(i0, std::true_type{}, acc, [&]() __attribute__((always_inline)) {
            if (i0 > 0) {
                __builtin_amdgcn_sched_barrier(0);
                tot[0] += acc[0];
                tot[1] += acc[1];
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        for (int i = i0 + 1; i < min(i0 + run, nk); ++i) slice(i, std::false_type{}, acc, [] {});
    }

    // Stage the 128 x 64 output tile (bias added, rounded) in LDS, rows of
    // kOutStride bytes: lane (l32, half) holds channels 32t + 8g + 4*half + (0..3)
    // of tile row 32*wave + l32.
    constexpr int kOutStride = kBN * 2 + 16;
    static_assert(kBM * kOutStride <= kLdsBytes, "output tile fits in the slice ring");
    lds_barrier();   // every wave is done with the slices
    {
        char* orow = smem + (32 * wave + l32) * kOutStride;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] = (FOLD ? tot[t][4 * g + e] + acc[t][4 * g + e] : acc[t][4 * g + e]) +
                           to_float<ET>((uint16_t)(bias[t][g][e >> 1] >> (16 * (e & 1))));
                u32x2 w;
                w[0] = pack2<ET>(v[0], v[1]);
                w[1] = pack2<ET>(v[2], v[3]);
                *(u32x2*)(orow + (32 * t + 8 * g + 4 * half) * 2) = w;
            }
    }
    lds_barrier();
    // 16 bytes per lane: chunk q = tid + 256j is tile row q / 8 + 32j, channels
    // n = n0 + 8 (q % 8) .. + 7 (inside one head, as head widths are multiples
    // of 8).  The channel offset is the same for all j; the row's batch and
    // token advance by 32 tokens per j.
    const int c8 = threadIdx.x & 7;
    const int n = n0 + 8 * c8;
    const int r0 = threadIdx.x >> 3;
    if (n < N) {
        const int yhw = P.yhw;
        uint16_t* __restrict__ Yc = P.y + bi * P.sy + chan_offset<YH>(n, L, yhw, 1.0f / (float)yhw);
        int b = (m0 + r0) / L, l = (m0 + r0) - b * L;   // token row m = b*L + l
#pragma unroll
        for (int j = 0; j < kBM * kBN / 8 / 256; ++j) {
            const int r = r0 + 32 * j;
            if (m0 + r < M) {
                const u32x4 v = *(const u32x4*)(smem + r * kOutStride + c8 * 16);
                const size_t row = YH ? ((size_t)b * (N / yhw) * L + l) * yhw : (size_t)(m0 + r) * N;
                *(u32x4*)(Yc + row) = v;
            }
            l += 32;
            while (l >= L) {
                l -= L;
                ++b;
            }
        }
    }
}

// The same product for grids of few tiles (few token rows): the reduced
// dimension is split over the workgroup's four waves instead of the tile.  Each
// wave multiplies the whole TM x TN tile over its own run of channels, through
// a private LDS ring of ST slices of 64 channels that no other wave touches,
// so the main loop has no workgroup barrier and a chain of K/64 slices becomes
// four chains of a quarter of the length; the partial tiles meet once in LDS.
// Bound by the latency of those chains and each CU's copy rate (a 64x64 tile of
// K = 1280 is 328 KB through one CU); with one slice per wave (ST = 1) two or
// three workgroups share a CU and cover each other's waits, which measured
// faster than deeper rings (512x1280x1280: 9.1 against 9.4 us with ST = 2).
template <int TM, int TN, int ST>
struct KsGeom {
    static constexpr int kSlice = (TM + TN) * kBK * 2;            // bytes
    static constexpr int kCopies = kSlice / 1024;                 // copy instructions per slice
    static constexpr int kOutRow = TN * 4 + 16;                   // bytes per row of a partial tile
    static constexpr int kRing = kRuns * ST * kSlice;
    static constexpr int kPart = kRuns * TM * kOutRow;
    static constexpr int kLds = kRing > kPart ? kRing : kPart;
    static_assert(kLds <= 160 * 1024 && TM % 32 == 0 && TN % 32 == 0, "geometry");
    static_assert(kCopies * (ST - 1) < 64, "copies in flight fit vmcnt");
};

// Wait until at most n (<= N) slices of this wave's copies are in flight.
template <int COPIES, int N>
__device__ __forceinline__ void ks_wait(int n) {
    if constexpr (N > 0) {
        if (n < N) {
            ks_wait<COPIES, N - 1>(n);
            return;
        }
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES * N) : "memory");
}

template <int ET, bool YH, int TM, int TN, int ST>
__global__ __launch_bounds__(256) void linear_ksplit_kernel(const LinGroup grp) {
    using G = KsGeom<TM, TN, ST>;
    constexpr int MB = TM / 32, NB = TN / 32, KS = kBK / 16;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = lane_id();
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int pi = (grp.n > 2 && tile >= grp.p[2].tile0) ? 2 : (grp.n > 1 && tile >= grp.p[1].tile0) ? 1 : 0;
    const LinProblem& P = grp.p[pi];
    const int bi = (tile - P.tile0) / P.per_batch;
    const int local = tile - P.tile0 - bi * P.per_batch;
    const uint16_t* __restrict__ X = P.x + bi * P.sx;
    const uint16_t* __restrict__ W = P.w + bi * P.sw;
    const int M = P.M, K = P.K, N = P.N, L = P.L;
    const int nmt = (M + TM - 1) / TM;
    const int mt = local % nmt;          // consecutive workgroups share the weight rows
    const int m0 = mt * TM;
    const int n0 = (local / nmt) * TN;

    // this wave's slices
    const int ns = (K + kBK - 1) / kBK;
    const int per = (ns + kRuns - 1) / kRuns;
    const int first = wave * per;
    const int count = max(0, min(per, ns - first));
    char* ring = smem + wave * (ST * G::kSlice);

    // Copy j moves chunk cch[j] / 8 of tile row r (x rows, then w rows); rows
    // past M or N repeat the last row (their outputs are never stored).
    const uint16_t* src[G::kCopies];
    int cch[G::kCopies];
#pragma unroll
    for (int j = 0; j < G::kCopies; ++j) {
        const int u = j * 64 + lane;
        const int r = u / 8;
        cch[j] = 8 * ((u % 8) ^ swz(r)) + first * kBK;
        src[j] = j * 64 < TM * 8 ? X + (size_t)min(m0 + r, M - 1) * K
                                 : W + (size_t)min(n0 + r - TM, N - 1) * K;
    }
    auto issue = [&](int i) __attribute__((always_inline)) {
        char* st = ring + (i % ST) * G::kSlice;
#pragma unroll
        for (int j = 0; j < G::kCopies; ++j)   // channels past K repeat the last chunk (zeroed below)
            __builtin_amdgcn_global_load_lds((const char*)(src[j] + min(cch[j] + i * kBK, K - 8)),
                                             (lds_void_t*)(st + j * 1024), 16, 0, 0);
    };

    int offx[KS], offw[KS];   // row l32, chunk 2s + half; rows 32 apart share the swizzle
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const int cpos = (2 * s + half) ^ swz(l32);
        offx[s] = (l32 * 8 + cpos) * 16;
        offw[s] = ((TM + l32) * 8 + cpos) * 16;
    }

    f32x16 acc[MB][NB];
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.0f;

#pragma unroll
    for (int i = 0; i < ST; ++i)
        if (i < count) issue(i);

    for (int i = 0; i < count; ++i) {
        ks_wait<G::kCopies, ST - 1>(count - 1 - i);
        const char* st = ring + (i % ST) * G::kSlice;
        u32x4 xf[MB][KS], wf[NB][KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
#pragma unroll
            for (int a = 0; a < MB; ++a) xf[a][s] = *(const u32x4*)(st + offx[s] + a * 32 * kBK * 2);
#pragma unroll
            for (int b = 0; b < NB; ++b) wf[b][s] = *(const u32x4*)(st + offw[s] + b * 32 * kBK * 2);
        }
        // the slot is read out: its next slice may be copied in
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (i + ST < count) issue(i + ST);
        const int kval = K - (first + i) * kBK;   // channels of this slice inside K
        if (kval < kBK) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
                if (8 * (2 * s + half) >= kval) {
#pragma unroll
                    for (int a = 0; a < MB; ++a) xf[a][s] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
                    for (int b = 0; b < NB; ++b) wf[b][s] = u32x4{0u, 0u, 0u, 0u};
                }
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int a = 0; a < MB; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[a][b] = mfma32x32x16<ET>(wf[b][s], xf[a][s], acc[a][b]);
    }

    // 16 bytes per lane: chunk q = tid + 256j is tile row q / (TN / 8), channels
    // n = n0 + 8 (q % (TN / 8)) .. + 7, the same n for every j
    constexpr int kCols = TN / 8;
    const int c8 = threadIdx.x % kCols;
    const int n = n0 + 8 * c8;
    u32x2 bias[2] = {u32x2{0u, 0u}, u32x2{0u, 0u}};
    if (P.bias && n < N) {
        bias[0] = *(const u32x2*)(P.bias + n);
        bias[1] = *(const u32x2*)(P.bias + n + 4);
    }

    // partial tiles: lane (l32, half) holds channels 32b + 8g + 4*half + (0..3)
    // of row 32a + l32
    __syncthreads();   // every wave is done with its ring
    {
        char* part = smem + wave * (TM * G::kOutRow);
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 v = {acc[a][b][4 * g], acc[a][b][4 * g + 1], acc[a][b][4 * g + 2],
                                     acc[a][b][4 * g + 3]};
                    *(f32x4*)(part + (32 * a + l32) * G::kOutRow + (32 * b + 8 * g + 4 * half) * 4) = v;
                }
    }
    __syncthreads();
    if (n >= N) return;
    const int yhw = P.yhw;
    uint16_t* __restrict__ Yc = P.y + bi * P.sy + chan_offset<YH>(n, L, yhw, 1.0f / (float)yhw);
#pragma unroll
    for (int j = 0; j < (TM * kCols + 256 - 1) / (256); ++j) {
        const int r = (threadIdx.x + 256 * j) / kCols;
        if (r < TM && m0 + r < M) {
            f32x4 lo = {0.0f, 0.0f, 0.0f, 0.0f}, hi = lo;
#pragma unroll
            for (int w = 0; w < kRuns; ++w) {
                const char* p = smem + w * (TM * G::kOutRow) + r * G::kOutRow + c8 * 32;
                lo += *(const f32x4*)p;
                hi += *(const f32x4*)(p + 16);
            }
            u32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const u32x2 bb = bias[e >> 1];
                const float b0 = to_float<ET>((uint16_t)bb[e & 1]);
                const float b1 = to_float<ET>((uint16_t)(bb[e & 1] >> 16));
                v[e] = e < 2 ? pack2<ET>(lo[2 * e] + b0, lo[2 * e + 1] + b1)
                             : pack2<ET>(hi[2 * e - 4] + b0, hi[2 * e - 3] + b1);
            }
            *(u32x4*)(Yc + row_base<YH>(m0 + r, L, N, yhw)) = v;
        }
    }
}

// tm x tn tiles of one batch item
long long tiles_of(const LinearArgs& a, int tm, int tn) {
    return ((long long)a.B * a.L + tm - 1) / tm * ((a.N + tn - 1) / tn);
}

template <int ET, bool XH, bool YH, bool FOLD>
hipError_t launch_t(const LinGroup& g, long long nblk, void* stream) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&linear_kernel<ET, XH, YH, FOLD>),
        hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((linear_kernel<ET, XH, YH, FOLD>), dim3((unsigned)nblk), dim3(256), kLdsBytes,
                       (hipStream_t)stream, g);
    return hipGetLastError();
}

template <int ET, bool XH, bool YH>
hipError_t launch_f(const LinGroup& g, long long nblk, bool fold, void* stream) {
    return fold ? launch_t<ET, XH, YH, true>(g, nblk, stream) : launch_t<ET, XH, YH, false>(g, nblk, stream);
}

// Number the TM x TN tiles of the group's products (tile0, per_batch, nnt);
// returns how many there are.
long long number_tiles(LinGroup& g, const LinearArgs* a, int tm, int tn) {
    long long nblk = 0;
    for (int i = 0; i < g.n; ++i) {
        g.p[i].nnt = (a[i].N + tn - 1) / tn;
        g.p[i].tile0 = (int)nblk;
        g.p[i].per_batch = (int)tiles_of(a[i], tm, tn);
        nblk += tiles_of(a[i], tm, tn) * a[i].batch;
        if (nblk > 0x7fffffff) return nblk;
    }
    return nblk;
}

template <int ET, bool YH, int TM, int TN, int ST>
hipError_t launch_ks(LinGroup& g, const LinearArgs* a) {
    using G = KsGeom<TM, TN, ST>;
    const long long nblk = number_tiles(g, a, TM, TN);
    if (nblk > 0x7fffffff) return hipErrorInvalidValue;
    auto k = linear_ksplit_kernel<ET, YH, TM, TN, ST>;
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, G::kLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(k, dim3((unsigned)nblk), dim3(256), G::kLds, (hipStream_t)a[0].stream, g);
    return hipGetLastError();
}

// The tile of the split-K kernel: 32 x 32 while those tiles fit the CUs once,
// 64 x 64 where rows past 32 would read the weights twice and there are tiles
// enough (two per CU), 32 x 64 between.  Measured (us, 32x32 / 32x64 / 64x64):
// 128x1280x1280 5.1 / 6.0 / 7+; 512x1280x1280 10.0 / 9.2 / 9.1; 36 products
// 48x1280x1280 - / 34.5 / 30.3; 36 of 64x640x640 12.2 / 9.5 / 10.3.
template <int ET, bool YH>
hipError_t launch_ksplit(LinGroup& g, const LinearArgs* a) {
    long long n32 = 0, n64 = 0, rows = 0;
    for (int i = 0; i < g.n; ++i) {
        n32 += tiles_of(a[i], 32, 32) * a[i].batch;
        n64 += tiles_of(a[i], 64, 64) * a[i].batch;
        rows = rows > g.p[i].M ? rows : g.p[i].M;
    }
    if (n32 <= 256) return launch_ks<ET, YH, 32, 32, 2>(g, a);
    if (rows > 32 && n64 >= 512) return launch_ks<ET, YH, 64, 64, 1>(g, a);
    return launch_ks<ET, YH, 32, 64, 1>(g, a);
}

template <int ET>
hipError_t launch_group_e(LinGroup& g, const LinearArgs* a) {
    const bool xh = a[0].x_heads, yh = a[0].y_heads;
    // Split K over the waves where 128-row tiles leave the chip idle (at most
    // 128 of them: half of the CUs) or mostly compute padding (at most 64 rows):
    // 512x1280x1280 (80 tiles) 12.1 -> 9.2 us, 768x1280x1280 (120) 12.1 -> 9.8,
    // 1280x640x640 (100) 7.7 -> 7.2, 36 products 32x1280x1280 31.3 -> 25.8.  From
    // there on the shared tiles are as fast or faster: 1024x1280x1280 (160 tiles)
    // 12.3 against 13.2, 3328x320x320 (130) 5.8 against 6.1, 36 products
    // 72x1280x1280 34.4 against 41.9.  Products split only past kSplitMinK
    // channels, where the shared tiles sum in the same order (FOLD): a row's bits
    // depend neither on its company in a launch nor on the other images of a batch.
    if (!xh) {
        long long tiles = 0;
        bool few_rows = true, may = true;
        for (int i = 0; i < g.n; ++i) {
            tiles += tiles_of(a[i], kBM, kBN) * a[i].batch;
            few_rows = few_rows && g.p[i].M <= 64;
            may = may && a[i].K > kSplitMinK;
        }
        if (may && (tiles <= 128 || few_rows))
            return yh ? launch_ksplit<ET, true>(g, a) : launch_ksplit<ET, false>(g, a);
    }
    const long long nblk = number_tiles(g, a, kBM, kBN);
    if (nblk > 0x7fffffff) return hipErrorInvalidValue;
    bool fold = false;
    for (int i = 0; i < g.n; ++i) fold = fold || a[i].K > kSplitMinK;
    void* s = a[0].stream;
    if (xh) return yh ? launch_f<ET, true, true>(g, nblk, fold, s) : launch_f<ET, true, false>(g, nblk, fold, s);
    return yh ? launch_f<ET, false, true>(g, nblk, fold, s) : launch_f<ET, false, false>(g, nblk, fold, s);
}

}  // namespace

long long linear_grid(int B, int L, int N) {
    // (the split-K kernel's smaller tiles are taken for at most 128 of these, or 64 rows)
    LinearArgs a{};
    a.B = B;
    a.L = L;
    a.N = N;
    return tiles_of(a, kBM, kBN);
}

hipError_t launch_linear_group(const LinearArgs* a, int n) {
    if (n < 1 || n > kMaxLinearProblems) return hipErrorInvalidValue;
    LinGroup g{};
    g.n = n;
    for (int i = 0; i < n; ++i) {
        if (a[i].dtype != a[0].dtype || a[i].x_heads != a[0].x_heads ||
            a[i].y_heads != a[0].y_heads || a[i].stream != a[0].stream || a[i].batch < 1)
            return hipErrorInvalidValue;
        LinProblem& p = g.p[i];
        p.x = (const uint16_t*)a[i].x;
        p.w = (const uint16_t*)a[i].w;
        p.bias = (const uint16_t*)a[i].bias;
        p.y = (uint16_t*)a[i].y;
        p.M = a[i].B * a[i].L;
        p.K = a[i].K;
        p.N = a[i].N;
        p.L = a[i].L;
        p.xhw = a[i].x_heads ? a[i].K / a[i].H : 1;
        p.yhw = a[i].y_heads ? a[i].N / a[i].H : 1;
        p.sx = a[i].sx;
        p.sw = a[i].sw;
        p.sy = a[i].sy;
    }
    return a[0].dtype == kF16 ? launch_group_e<kF16>(g, a) : launch_group_e<kBF16>(g, a);
}

hipError_t launch_linear(const LinearArgs& a) { return launch_linear_group(&a, 1); }

}  // namespace sdattn
