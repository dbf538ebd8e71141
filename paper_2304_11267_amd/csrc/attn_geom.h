// attn_geom.h -- the tiled attention kernel's workgroup geometries and the choice
// among them (attn_fwd_kernel.h has the kernel).  Plain C++, no device code.
#pragma once

namespace sdattn {

// Workgroup geometries (the GEO template argument): rows of queries per
// workgroup and keys per LDS tile.
constexpr int kGeoSmall = 0;           // 64 rows, 64-key tiles
constexpr int kGeoNormal = 1;          // 128 rows, 64-key tiles
constexpr int kGeoBig = 2;             // 256 rows, 64-key tiles (QB = 2 only)
constexpr int kGeoQuarter = 3;         // 64 rows, keys split four ways, 64-key tiles
constexpr int kGeoPair = 4;            // kGeoNormal without the streaming loop's third buffer
constexpr int kMaxLds = 160 * 1024;
constexpr int kQuarterMinKeys = 512;   // shortest key sequence given to kGeoQuarter
constexpr int kBigMinKeys = 1024;      // and to kGeoBig
constexpr int kCus = 256;

// QB = 32-row query blocks per wave.  With QB = 2 every K and V^T operand
// read from LDS feeds two MFMAs (half the LDS traffic per flop) and each wave
// carries two independent MFMA / softmax chains; the register budget is then
// sized for two waves per SIMD.
//
// kGeoSmall halves the query waves of a workgroup (64 query rows instead of
// 128), for calls whose 128-row blocks would leave CUs idle (the 32x32 and
// 16x16 levels).  kGeoBig doubles them (256 rows, eight waves): each K/V tile
// then serves twice the queries.
// kGeoQuarter keeps kGeoSmall's 64 rows but splits the keys four ways
// instead of two (eight waves), for small grids whose LDS would otherwise
// leave one wave per SIMD: two waves then share each SIMD and hide each
// other's MFMA and exponential latencies.  Its tiles carry no constant
// block (the LDS holds four splits' double buffers), so l comes from v_dot2.
// kGeoPair is for widths (D = 56, 64) whose streaming ring fills a CU's LDS with
// one 128-row workgroup, four waves: with two buffers a CU holds two.
template <int D, int GEO = kGeoNormal>
struct Geom {
    static constexpr int QB = D <= 64 ? 2 : 1;
    static constexpr bool kBig = GEO == kGeoBig;
    static constexpr bool kQuarter = GEO == kGeoQuarter;
    static constexpr int kKS = kQuarter ? 4 : 2;              // key splits
    static constexpr int kTK = 64;                            // keys per LDS tile
    static constexpr int kQW = kBig ? 4 : (GEO == kGeoSmall || kQuarter ? 2 : 4) / QB;   // query waves
    static constexpr int kBQ = 32 * QB * kQW;                 // query rows per workgroup
    static constexpr int kWaves = kKS * kQW;                  // times the key splits
    static constexpr int kThreads = kWaves * 64;
    static constexpr int DK = (D + 15) / 16;                  // 16-deep k steps of Q K^T
    static constexpr int DN = (D + 31) / 32;                  // 32-row d tiles of O^T
    // At most 16 rows of O^T left over from whole 32-row tiles: they go through
    // one sparse MFMA per 32 keys instead of two dense ones (step32's O^T).
    static constexpr bool kSparse = D % 32 == 8 || D % 32 == 16;
    static constexpr int DD = kSparse ? DN - 1 : DN;          // dense d tiles
    static constexpr bool kOnes = (D % 32 == 8 || D % 32 == 24) && !kQuarter;   // padding rows carry the row sum
    static constexpr int kTileBytes = kTK * D * 2;            // one K or V tile
    static constexpr int kChunks = kTileBytes / 1024;         // 1 KiB wave copies per tile
    static constexpr int kBufBytes = 2 * kTileBytes;          // K, V
    static constexpr int kConstBytes = kOnes ? kTileBytes : 0;   // the constant block
    // The streaming loop (stream_tiles) works on two tiles at once and takes a
    // ring of three buffers per key split (five where a workgroup fills a CU and
    // meets only every second tile); the other loop takes two.  It needs two
    // query blocks a wave (each LDS operand then feeds two MFMAs; with one the LDS
    // is as busy as the matrix core).  16 heads of as many rows as keys, the other
    // loop / this one, us: 4096 keys D = 32 49.9 / 47.4, D = 40 56.6 / 52.6, D = 64
    // 82.1 / 75.2; 2048 keys D = 64 26.8 / 23.3, D = 48 20.8 / 18.8; 2048 rows of 300
    // keys D = 40 8.3 / 7.1.  Not for D = 48 in 256 rows, the one width that it
    // measured slower at (why, is not known): 4096 keys 59.7 / 60.4, 2048 32.1 / 33.0,
    // with statistics 65.2 / 66.2.  The four key splits of kGeoQuarter leave it too few
    // tiles each (1024 keys D = 40 9.5 / 10.1).
    static constexpr int kRoom = kMaxLds - 64 - kConstBytes;
    static constexpr bool kStream = QB == 2 && !kQuarter && GEO != kGeoPair && !(kBig && D == 48) &&
                                    kKS * 3 * kBufBytes <= kRoom;
    static constexpr int kSlots = !kStream ? 2 : kBig && kKS * 5 * kBufBytes <= kRoom ? 5 : 3;
    static constexpr int kStep = kSlots == 5 ? 2 : 1;         // tiles between two barriers of the streaming loop
    static constexpr int kHalfBytes = kSlots * kBufBytes;
    static constexpr int kConst = kKS * kHalfBytes;
    static constexpr int kRegs = 16 * DN - (kSparse ? 8 : 0);   // O^T registers with rows of O in them
    static constexpr int kMergeFloats = QB * (kRegs * 64 + 3 * 64);   // one wave's O^T, m, max, l
    static constexpr int kMergeBytes = (kKS - 1) * kQW * kMergeFloats * 4;
    static constexpr int kTiles = kConst + kConstBytes;
    static constexpr int kUsed = kTiles > kMergeBytes ? kTiles : kMergeBytes;
    static constexpr int kVote = kStream ? kUsed : 0;         // overflow votes: their own words, or the idle first tile
    static constexpr int kLdsBytes = kUsed + (kStream ? 64 : 0);
    static constexpr bool kFits = D >= 32 && D % 8 == 0 && kLdsBytes <= kMaxLds && (!kBig || QB == 2) &&
                                  (GEO != kGeoPair || D == 56 || D == 64);
    // Waves per SIMD the register budget is sized for: two (256 registers
    // each) when the LDS lets enough workgroups share a CU, else one, which
    // leaves a wave up to 512 registers (the matrix-core registers then take
    // what would otherwise spill to scratch) at no cost in occupancy.  (The
    // streaming loop keeps 256 also for the odd waves of three workgroups a CU.)
    static constexpr int kWgPerCu = kLdsBytes <= kMaxLds ? kMaxLds / kLdsBytes : 1;
    static constexpr int kWavesPerSimd = kWgPerCu * kWaves >= (kStream ? 5 : 8) ? 2 : 1;
};

// The geometry of a call over `heads` (batch, head) pairs.  What counts is how
// often the fullest CU starts over: a grid of one workgroup more than the CUs
// takes twice the time of one that just covers them, however few rows are left
// for the second round, and rows past Lq cost as much as others.
template <int D>
int pick_geometry(long long heads, int Lq, int Lk) {
    auto rounds = [&](int rows) { return (heads * ((Lq + rows - 1) / rows) + kCus - 1) / kCus; };
    const long long r128 = rounds(128);
    // 64 rows where they take no more rounds than 128 (a round of them is 5 to 20 %
    // shorter), the keys split four ways (more waves per SIMD) once every split has
    // two tiles.  Else 128: D = 40, 1024 keys, 320 64-row blocks of 20 heads 14.5 us in two
    // rounds (four splits 12.2) against 10.3 in one round of 160; D = 160 with
    // statistics 35.6 against 25.3.
    if (rounds(64) <= r128) {
        if constexpr (Geom<D, kGeoQuarter>::kFits) {
            if (Lk >= kQuarterMinKeys) return kGeoQuarter;
        }
        return kGeoSmall;
    }
    // 256 rows where that halves the rounds, and two of: to one; 128 rows would stream
    // alone on their CU; a long key loop (a tile then serves twice the rows, and a
    // workgroup meets half as often).  128 / 256 rows, us: D = 40, 9 heads of 4096 rows (2
    // rounds / 1) 47.1 / 43.1 at 4096 keys, 15.6 / 15.4 at 1024, 10.4 / 10.5 at 512; D = 48,
    // 32 heads (4 / 2) 63.4 / 66.2 at 2048; 24 heads (3 / 2) of D = 40 79.8 / 95.1.  D = 64
    // against kGeoPair: 9 heads 13.7 / 13.4 at 300 keys, 41.8 / 35.5 at 2048; 32 heads 26.1 /
    // 28.0 and 86.9 / 83.9
    if constexpr (Geom<D, kGeoBig>::kFits) {
        const long long r256 = rounds(256);
        const int points = (r256 == 1) + Geom<D, kGeoPair>::kFits + (Lk >= kBigMinKeys);
        if (r128 == 2 * r256 && points >= 2) return kGeoBig;
    }
    // Past one round two workgroups on a CU beat the streaming loop alone on it
    // (kGeoNormal / kGeoPair / kGeoBig, us, D = 64): 24 heads of 4096 rows 68.7 / 66.8 / 76.7
    // at 2048 keys, 26.1 / 21.9 / 26.8 at 300; 384 heads of 128 rows 30.4 / 26.7 / 42.6 at
    // 1024.  In one round it is the slower loop: 14.7 / 16.1
    if constexpr (Geom<D, kGeoPair>::kFits) {
        if (r128 > 1) return kGeoPair;
    }
    return kGeoNormal;
}

}  // namespace sdattn
