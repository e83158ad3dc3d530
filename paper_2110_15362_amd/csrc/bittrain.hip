// libbittrain: BitTrain's sparse bitmap activation codec as HIP kernels for
// CDNA4 (gfx950, wave64).  See include/bittrain.h for the contract.
//
// Section 3.2 of the paper defines the format (a bit per element plus the
// non-zero elements in index order); Algorithm 1 builds it with a sequential
// append loop and Algorithm 2 undoes it with a running counter j.  Both loops
// carry one dependency: the position of an element's value is the number of
// non-zero elements before it.  On a GPU that is an exclusive prefix sum over
// the non-zero predicate, and the kernels below compute it in ONE pass over the
// data so that the tensor is read from HBM exactly once:
//
//   lane    16-byte loads; per-lane non-zero mask by integer compare
//   wave    packed DPP prefix sum of the per-lane popcounts (no LDS, no barrier)
//   block   four wave totals through LDS
//   grid    per-tile counts published in the workspace; one extra wave turns them
//           into per-tile prefixes; a wave polls only the prefix of its own tile
//
// A codec launch has one workgroup per 32 KiB tile, plus one, whose first wave is the
// scanner; launches on small tensors have no scanner, and smaller tiles.  No workgroup
// depends on another for progress: a workgroup whose prefix has not come after a bounded
// number of polls counts the elements before its tile itself, from the input (compression)
// or from the bitmap (restoration), so the order in which the hardware starts the workgroups
// does not matter.  A workgroup ends with its stores on their way; it never waits for them
// to land.
//
// There is no matrix contraction anywhere, so no MFMA: the path is bound by HBM
// bandwidth and everything here is about moving each byte once, coalesced, and
// about keeping the memory system busy while prefixes are on their way.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "bittrain.h"

namespace {

constexpr int kWaveSize = 64;
constexpr int kWaves = 4;                 // waves per block
constexpr int kBlock = kWaveSize * kWaves;
constexpr int kRows = 8;                  // 16-byte loads per lane per tile: of the tile index, of batches and of all but small tensors
constexpr int kVecBytes = 16;
// LDS of a compressing workgroup: what eight of them on a compute unit leave each other of its 160 KiB, less the
// words beside the staging area.
constexpr int kStageBytes = 160 * 1024 / 8 - 64;
#ifndef BT_RELU_ROWS
#define BT_RELU_ROWS 1
#endif
constexpr int kReluRows = BT_RELU_ROWS;   // 16-byte vectors per lane in the ReLU-backward stream

// Workgroups per compute unit (= waves per SIMD) the codec kernels are built for: eight, i.e. at
// most 64 vector registers per lane.
#ifndef BT_COMPRESS_OCC
#define BT_COMPRESS_OCC 8
#endif
#ifndef BT_DECOMPRESS_OCC
#define BT_DECOMPRESS_OCC 8
#endif
constexpr int kCompressOcc = BT_COMPRESS_OCC;
constexpr int kDecompressOcc = BT_DECOMPRESS_OCC;

// ---- workspace layout -----------------------------------------------------------------
// Header (uint32 words), then one 6 KiB block per 256 slots.
constexpr int kHdrCalls = 0;     // calls completed on this workspace
constexpr int kHdrEntries = 1;   // bits 0-30: slots of the previous call that used the entries (what it left behind in the other
                                 // copy); bit 31: the copy that the next such call uses
constexpr int kHdrError = BT_WS_ERROR_WORD;           // set if a wait was given up
constexpr int kHdrSpinLimit = BT_WS_WAIT_LIMIT_WORD;  // scanner passes before its wait is given up; 0: kSpinLimit
constexpr int kHdrWide = BT_WS_WIDE_WORD;             // non-zero: the one-tensor scanner writes 8-byte entries only
constexpr int kHdrPatience = BT_WS_PATIENCE_WORD;     // polls before a workgroup counts what precedes its tile itself; 0: kPatience
[[maybe_unused]] constexpr int kHdrMute = BT_WS_MUTE_WORD;      // instrumented build; non-zero: tiles are not told their prefixes
constexpr size_t kHeaderBytes = 256;
// Block of 256 slots, two copies c = 0, 1 of everything:
//   [1024*c, 1024*c + 1024)            uint32 count + 1 of each slot, written by the slot's workgroup
//   [2048 + 2048*c, 2048*c + 4096)     uint64 prefix + 1 of each slot, written by the scanner
// 0 means "not published yet".  A call uses one copy and zeroes what the
// previous call left in the other copy, so the copy the next call uses is clean
// when it starts and no clearing launch is ever needed.  The layout depends only on the
// slot number, never on the size of the workspace or of the call.
constexpr int kSlotsPerBlock = 256;
constexpr size_t kBlockBytes = 6144;
constexpr uint32_t kSpinLimit = 1u << 20; // scanner passes before its wait is given up
constexpr uint32_t kPatience = 1u << 12;  // polls before a workgroup counts what precedes its tile itself instead of waiting on
#ifndef BT_SCANNER_SLEEP
#define BT_SCANNER_SLEEP 1
#endif
// Launches of up to this many slots store a dense output before the prefix is there (element bytes S; see compress_kernel).
template <int S> constexpr uint32_t kDenseEarlySlots = S == 2 ? 1280 : 1000;
constexpr int kScannerSleep = BT_SCANNER_SLEEP;   // pause between two polls, in units of 64 clocks

// S: element bytes; R: rows (16-byte loads) per lane per tile; W: waves of the workgroup that a tile belongs to.
template <int S, int R = kRows, int W = kWaves> struct Geo {
    static constexpr int E = kVecBytes / S;          // elements per lane per load
    static constexpr int G = 32 / E;                 // lanes that share a bitmap word
    static constexpr int WPR = kWaveSize / G;        // bitmap words per row
    static constexpr int ROW = kWaveSize * E;        // elements per wave-wide load
    static constexpr int WAVE = R * ROW;             // elements per wave per tile
    static constexpr int PHASE = R < 4 ? R : 4;      // rows that are compacted / expanded through LDS at a time
    static constexpr int TILE = W * WAVE;            // elements per tile
    static constexpr int TILE_WORDS = TILE / 32;     // bitmap words per tile
    static constexpr int WAVE_WORDS = TILE_WORDS / W;      // of which a wave's quarter of the tile has this many
    static constexpr int QPL = WAVE_WORDS > kWaveSize ? WAVE_WORDS / kWaveSize : 1;   // and a lane reads this many (of a quarter)
    static constexpr int WPL = TILE_WORDS > kWaveSize ? TILE_WORDS / kWaveSize : 1;   // or this many (of the whole tile)
    static constexpr int LDS_WAVE = PHASE * ROW * S + 2 * kVecBytes;  // restoration's staging bytes per wave: the rows of a phase, the
                                                                          // shift to a 16-byte boundary, and what a read past the last value may touch
    static constexpr int LDS_TILE = PHASE * W * kWaveSize * kVecBytes + 2 * kVecBytes;      // and per workgroup, where its waves stage together
    static constexpr int STAGE = TILE * S <= kStageBytes - kVecBytes ? TILE * S : kStageBytes - kVecBytes;   // compression: bytes of a tile's
                                                                          // values that fit LDS together (then a vector nobody reads)
    static constexpr int RPM = 32 / E;               // rows whose E-bit lane masks share one register
    static constexpr int MW = (R + RPM - 1) / RPM;   // registers that hold a lane's masks
    static_assert(R % PHASE == 0 && PHASE % 2 == 0, "rows are scanned two to a register");
};

// ---- wave-level primitives (all 64 lanes must be active) ---------------------

#define BT_DPP(old, src, ctrl, rmask, bound) \
    ((uint32_t)__builtin_amdgcn_update_dpp((int)(old), (int)(src), (ctrl), (rmask), 0xf, (bound)))

// Inclusive prefix sum over the 64 lanes.  Four shift-and-add steps inside each
// row of 16 lanes (lanes shifted in from outside the row read 0), then the last
// lane of row 0 / row 2 is added to row 1 / row 3, then lane 31 to rows 2 and 3.
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x) {
    x += BT_DPP(0, x, 0x111, 0xf, true);   // row_shr:1
    x += BT_DPP(0, x, 0x112, 0xf, true);   // row_shr:2
    x += BT_DPP(0, x, 0x114, 0xf, true);   // row_shr:4
    x += BT_DPP(0, x, 0x118, 0xf, true);   // row_shr:8
    x += BT_DPP(0, x, 0x142, 0xa, false);  // row_bcast:15 into rows 1 and 3
    x += BT_DPP(0, x, 0x143, 0xc, false);  // row_bcast:31 into rows 2 and 3
    return x;
}

// Inclusive running maximum over the 64 lanes, in the same steps.
__device__ __forceinline__ uint32_t wave_inclusive_max(uint32_t x) {
    x = max(x, BT_DPP(0, x, 0x111, 0xf, true));
    x = max(x, BT_DPP(0, x, 0x112, 0xf, true));
    x = max(x, BT_DPP(0, x, 0x114, 0xf, true));
    x = max(x, BT_DPP(0, x, 0x118, 0xf, true));
    x = max(x, BT_DPP(0, x, 0x142, 0xa, false));
    x = max(x, BT_DPP(0, x, 0x143, 0xc, false));
    return x;
}

// The lanes' numbers added up, in 64 bits.  (By DPP, in two halves: shuffles would keep an address per step in a register,
// which compression cannot spare.)
__device__ __forceinline__ uint64_t wave_total_of(uint32_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(x & 0xffffu), 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(x >> 16), 63);
    return ((uint64_t)hi << 16) + lo;
}

// OR over each aligned group of G lanes (G = 4, 8 or 16); every lane gets the result.
template <int G> __device__ __forceinline__ uint32_t group_or(uint32_t x) {
    x |= BT_DPP(0, x, 0xB1, 0xf, true);       // quad_perm [1,0,3,2]: lane ^ 1
    x |= BT_DPP(0, x, 0x4E, 0xf, true);       // quad_perm [2,3,0,1]: lane ^ 2
    if (G >= 8) x |= BT_DPP(0, x, 0x141, 0xf, true);   // row_half_mirror: lane i <-> 7 - i
    if (G == 16) x |= BT_DPP(0, x, 0x140, 0xf, true);  // row_mirror: lane i <-> 15 - i
    return x;
}

// A workgroup barrier that orders LDS traffic only.  (__syncthreads() also waits for every global load
// and store of the wave, which would make a wave that has the next tile's loads in flight wait for them.)
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The lane's number, computed where it is needed instead of kept in a register up to there.
__device__ __forceinline__ int lane_number() {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// Order LDS traffic between the lanes of one wave (no block barrier involved).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- per-lane helpers -----------------------------------------------------------

// Bulk data is touched exactly once per call, so most of it is moved with the
// "non-temporal" hint: it then does not displace what the caches hold.  Measured per
// kernel on MI355X (fp32, 25.7 M elements, cold / warm microseconds):
//   compress    plain 38.1/31.3   nt loads 34.2/32.8   nt stores 35.0/30.0   both 33.3/31.3
//   decompress  plain 35.6/27.6   nt loads 36.3/32.8   nt stores 34.4/27.3   both 35.0/34.2
//   relu bwd    plain 37.2        nt loads 36.6        nt stores 35.4        both 34.7
// so compress and the ReLU stream of large gradients use both hints (their input is dead after the call:
// Algorithm 1 ends by giving the dense tensor up), decompress only the store hint.
typedef uint32_t bt_u4 __attribute__((ext_vector_type(4)));
typedef uint32_t bt_u2 __attribute__((ext_vector_type(2)));
template <bool NT> __device__ __forceinline__ uint4 stream_load(const uint4 *p) {
    if (NT) {
        const bt_u4 v = __builtin_nontemporal_load(reinterpret_cast<const bt_u4 *>(p));
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    return *p;
}
template <bool NT> __device__ __forceinline__ void stream_store(uint4 *p, const uint4 v) {
    if (NT) {
        bt_u4 t;
        t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
        __builtin_nontemporal_store(t, reinterpret_cast<bt_u4 *>(p));
    } else {
        *p = v;
    }
}
constexpr bool kCompressNtLoad = true, kCompressNtStore = true;
constexpr bool kDecompressNtLoad = false, kDecompressNtStore = true;
constexpr bool kReluNtStore = true;

// Bit j set <=> element j of the 16-byte vector has a non-zero bit pattern.
// min(bits, 1) instead of a compare: a compare result lives in a scalar register
// pair, and 8 rows x 4..8 compares in flight exhaust the scalar registers.
template <int S> __device__ __forceinline__ uint32_t nonzero_mask(const uint4 v) {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
    if (S == 8) {
        m = min(d[0] | d[1], 1u) | (min(d[2] | d[3], 1u) << 1);
    } else if (S == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) m |= min(d[i], 1u) << i;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            m |= min(d[i] & 0xffffu, 1u) << (2 * i);
            m |= min(d[i] >> 16, 1u) << (2 * i + 1);
        }
    }
    return m;
}

// Which elements of the 16-byte vector are stored.  KEEP = kKeepNonZero: Algorithm 1's
// test (non-zero bit pattern).  Otherwise activation pruning (Section 4.3) followed by
// that test, in one pass: an element survives pruning where its value exceeds the
// threshold, compared in single precision after widening (exact for half and
// bfloat16; a double is compared in double precision with `threshold_f64`; a NaN
// exceeds nothing), and is then stored if its bit pattern is non-zero (a +0.0 that
// survives a negative threshold is still a zero for Algorithm 1).
enum { kKeepNonZero = 0, kKeepAboveF32 = 1, kKeepAboveF16 = 2, kKeepAboveBF16 = 3, kKeepAboveF64 = 4 };
template <int S, int KEEP>
__device__ __forceinline__ uint32_t keep_mask(const uint4 v, const float threshold, const double threshold_f64) {
    if (KEEP == kKeepNonZero) return nonzero_mask<S>(v);
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
    if (KEEP == kKeepAboveF64) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            m |= (__builtin_bit_cast(double, bt_u2{d[2 * i], d[2 * i + 1]}) > threshold_f64 ? 1u : 0u) << i;
    } else if (KEEP == kKeepAboveF32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) m |= (__uint_as_float(d[i]) > threshold ? 1u : 0u) << i;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float lo, hi;
            if (KEEP == kKeepAboveBF16) {
                lo = __uint_as_float(d[i] << 16);
                hi = __uint_as_float(d[i] & 0xffff0000u);
            } else {
                lo = (float)__builtin_bit_cast(_Float16, (uint16_t)(d[i] & 0xffffu));
                hi = (float)__builtin_bit_cast(_Float16, (uint16_t)(d[i] >> 16));
            }
            m |= (lo > threshold ? 1u : 0u) << (2 * i);
            m |= (hi > threshold ? 1u : 0u) << (2 * i + 1);
        }
    }
    return m & nonzero_mask<S>(v);
}

// 16 bytes at element index e0 of a buffer of n > 0 elements; elements at or beyond n
// read as 0.  Branch-free: every address is clamped into the buffer, then selected.
template <int S> __device__ __forceinline__ uint4 load_vec_guarded(const void *base, uint64_t e0, uint64_t n) {
    uint32_t d[4] = {0, 0, 0, 0};
    if (S == 8) {
        const uint64_t *p = static_cast<const uint64_t *>(base);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint64_t e = e0 + j;
            const uint64_t v = p[e < n ? e : n - 1];
            d[2 * j] = e < n ? (uint32_t)v : 0u;
            d[2 * j + 1] = e < n ? (uint32_t)(v >> 32) : 0u;
        }
    } else if (S == 4) {
        const uint32_t *p = static_cast<const uint32_t *>(base);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t e = e0 + j;
            const uint32_t v = p[e < n ? e : n - 1];
            d[j] = e < n ? v : 0u;
        }
    } else {
        const uint16_t *p = static_cast<const uint16_t *>(base);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint64_t e = e0 + j;
            const uint32_t v = p[e < n ? e : n - 1];
            d[j >> 1] |= (e < n ? v : 0u) << (16 * (j & 1));
        }
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

template <int S> __device__ __forceinline__ void store_vec_guarded(void *base, uint64_t e0, uint64_t n, const uint4 v) {
    constexpr int E = Geo<S>::E;
    if (e0 + E <= n) {
        *reinterpret_cast<uint4 *>(static_cast<char *>(base) + e0 * S) = v;
        return;
    }
    if (e0 >= n) return;      // (of a whole wave but one lane at most: what follows is skipped as one)
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    if (S == 8) {
        uint64_t *p = static_cast<uint64_t *>(base);
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (e0 + j < n) p[e0 + j] = ((uint64_t)d[2 * j + 1] << 32) | d[2 * j];
    } else if (S == 4) {
        uint32_t *p = static_cast<uint32_t *>(base);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (e0 + j < n) p[e0 + j] = d[j];
    } else {
        uint16_t *p = static_cast<uint16_t *>(base);
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (e0 + j < n) p[e0 + j] = (uint16_t)(d[j >> 1] >> (16 * (j & 1)));
    }
}

// The E bitmap bits of the 16-byte vector that starts at element e0 (e0 % E == 0).
// Words at or beyond n_words read as 0, bits at or beyond n are cleared.
template <int S>
__device__ __forceinline__ uint32_t bitmap_bits(const uint32_t *bitmap, uint64_t e0, uint64_t n, uint64_t n_words) {
    constexpr int E = Geo<S>::E;
    const uint64_t w = e0 >> 5;
    uint32_t word = (w < n_words) ? bitmap[w] : 0u;
    uint32_t m = (word >> (uint32_t)(e0 & 31)) & ((1u << E) - 1u);
    if (e0 + E > n) m &= (e0 < n) ? ((1u << (uint32_t)(n - e0)) - 1u) : 0u;
    return m;
}

// ---- the tensors of a call ------------------------------------------------------------------
//
// A call works on one tensor or (the batched calls) on a list.  The tensors' tiles are laid end to
// end in a numbering of SLOTS (= workspace entries): a call on one tensor has slot == tile,
// in a batched call a tensor's first tile has the slot behind the previous tensor's last one.  Prefixes restart
// at 0 with every tensor and each tensor's total goes to its nnz.  The kernels see the call through a
// small interface (slots, at, and the per-tensor pointers) that the
// single-tensor and the batched argument structs both provide; the per-tensor pointers of a
// batched call travel as kernel arguments and are read with scalar loads.

struct Slot {
    uint32_t item;   // tensor of the call
    uint32_t tile;   // tile inside that tensor
};

constexpr int kMaxBatchDecompress = BT_MAX_BATCH;   // tensors per launch: what keeps the kernel arguments under 4 KiB
constexpr int kMaxBatchCompress = 52;

template <int MAXB> struct BatchLayout {
    uint32_t coarse[8];                       // start[0], start[8], ..., start[56]
    uint32_t start[(MAXB + 8) / 8 * 8];       // first slot of each tensor (an empty one: that of the next); from `count` on the end of the last one
    uint32_t count;
    static_assert(MAXB <= 64, "two steps of eight");
    // The tensor of a slot (slot < start[count]): every workgroup looks it up before it can ask for anything, so
    // in two steps of eight entries that each come with one scalar load, where halving takes six loads in a row.
    // (With the scanner's slot ranges kept in registers, see scan_counts: the 49 fp32 activations of a ResNet-50 at
    // batch 64 restore in 601 us instead of 621 and compress in 539 instead of 548.)
    __device__ __forceinline__ Slot at(const uint32_t slot) const {
        // (slot numbers are below 2^31, so the sign of a difference compares them: scalar arithmetic, where a
        // comparison's result would go through vector registers)
        uint32_t block = 0, item;
#pragma unroll
        for (int i = 1; i < 8; ++i) block += (coarse[i] - 1u - slot) >> 31;
        item = 8u * block;
#pragma unroll
        for (int i = 1; i < 8; ++i) item += (start[8u * block + i] - 1u - slot) >> 31;
        return Slot{item, slot - start[item]};
    }
};

struct CompressOne {
    static constexpr bool kMany = false;      // several tensors in one launch
    static constexpr bool kTotals = true;     // every tensor's number of values is asked for
    const void *in_;
    uint64_t n_;
    uint32_t *bitmap_;
    void *values_;
    uint64_t cap_;
    uint64_t *nnz_;
    uint64_t *index_;
    void *dense_;
    uint32_t tiles_;
    __device__ __forceinline__ uint32_t slots() const { return tiles_; }
    __device__ __forceinline__ Slot at(uint32_t slot) const { return Slot{0, slot}; }
    __device__ __forceinline__ const void *in(uint32_t) const { return in_; }
    __device__ __forceinline__ uint64_t n(uint32_t) const { return n_; }
    __device__ __forceinline__ uint32_t *bitmap(uint32_t) const { return bitmap_; }
    __device__ __forceinline__ void *values(uint32_t) const { return values_; }
    __device__ __forceinline__ uint64_t cap(uint32_t) const { return cap_; }
    __device__ __forceinline__ uint64_t *nnz(uint32_t) const { return nnz_; }
    __device__ __forceinline__ uint64_t *index(uint32_t) const { return index_; }
    __device__ __forceinline__ void *dense(uint32_t) const { return dense_; }
};

struct CompressMany {
    static constexpr bool kMany = true;      // several tensors in one launch
    static constexpr bool kTotals = true;
    BatchLayout<kMaxBatchCompress> lay;
    const void *in_[kMaxBatchCompress];
    uint64_t n_[kMaxBatchCompress];
    uint32_t *bitmap_[kMaxBatchCompress];
    void *values_[kMaxBatchCompress];
    uint64_t cap_[kMaxBatchCompress];
    uint64_t *nnz_[kMaxBatchCompress];
    uint64_t *index_[kMaxBatchCompress];
    void *dense_[kMaxBatchCompress];
    __device__ __forceinline__ uint32_t count() const { return lay.count; }
    __device__ __forceinline__ uint32_t start(uint32_t i) const { return lay.start[i]; }
    __device__ __forceinline__ uint32_t slots() const { return lay.start[lay.count]; }
    __device__ __forceinline__ Slot at(uint32_t slot) const { return lay.at(slot); }
    __device__ __forceinline__ const void *in(uint32_t i) const { return in_[i]; }
    __device__ __forceinline__ uint64_t n(uint32_t i) const { return n_[i]; }
    __device__ __forceinline__ uint32_t *bitmap(uint32_t i) const { return bitmap_[i]; }
    __device__ __forceinline__ void *values(uint32_t i) const { return values_[i]; }
    __device__ __forceinline__ uint64_t cap(uint32_t i) const { return cap_[i]; }
    __device__ __forceinline__ uint64_t *nnz(uint32_t i) const { return nnz_[i]; }
    __device__ __forceinline__ uint64_t *index(uint32_t i) const { return index_[i]; }
    __device__ __forceinline__ void *dense(uint32_t i) const { return dense_[i]; }
};
static_assert(sizeof(CompressMany) <= 3840, "kernel arguments of a batched compression");

struct DecompressOne {
    static constexpr bool kMany = false;      // several tensors in one launch
    static constexpr bool kTotals = false;
    const uint32_t *bitmap_;
    const void *values_;
    uint64_t cap_;
    const uint64_t *index_;
    uint64_t n_;
    void *out_;
    uint32_t tiles_;
    __device__ __forceinline__ uint32_t slots() const { return tiles_; }
    __device__ __forceinline__ Slot at(uint32_t slot) const { return Slot{0, slot}; }
    __device__ __forceinline__ const uint32_t *bitmap(uint32_t) const { return bitmap_; }
    __device__ __forceinline__ const void *values(uint32_t) const { return values_; }
    __device__ __forceinline__ uint64_t cap(uint32_t) const { return cap_; }
    __device__ __forceinline__ const uint64_t *tile_index(uint32_t) const { return index_; }
    __device__ __forceinline__ uint64_t n(uint32_t) const { return n_; }
    __device__ __forceinline__ void *out(uint32_t) const { return out_; }
};

struct DecompressMany {
    static constexpr bool kMany = true;      // several tensors in one launch
    static constexpr bool kTotals = false;
    BatchLayout<kMaxBatchDecompress> lay;
    const uint32_t *bitmap_[kMaxBatchDecompress];
    const void *values_[kMaxBatchDecompress];
    uint64_t cap_[kMaxBatchDecompress];
    const uint64_t *index_[kMaxBatchDecompress];
    uint64_t n_[kMaxBatchDecompress];
    void *out_[kMaxBatchDecompress];
    __device__ __forceinline__ uint32_t slots() const { return lay.start[lay.count]; }
    __device__ __forceinline__ Slot at(uint32_t slot) const { return lay.at(slot); }
    __device__ __forceinline__ const uint32_t *bitmap(uint32_t i) const { return bitmap_[i]; }
    __device__ __forceinline__ const void *values(uint32_t i) const { return values_[i]; }
    __device__ __forceinline__ uint64_t cap(uint32_t i) const { return cap_[i]; }
    __device__ __forceinline__ const uint64_t *tile_index(uint32_t i) const { return index_[i]; }
    __device__ __forceinline__ uint64_t n(uint32_t i) const { return n_[i]; }
    __device__ __forceinline__ void *out(uint32_t i) const { return out_[i]; }
};
static_assert(sizeof(DecompressMany) <= 3840, "kernel arguments of a batched restoration");

// ---- grid prefix ---------------------------------------------------------------------------
//
// The position of a tile's first value is the number of non-zero elements in all
// tiles before it (Algorithm 1 appends in index order; Algorithm 2's counter j).
// Tiles do not talk to each other.  Each tile's workgroup publishes its count in the
// workspace; ONE extra workgroup (workgroup 0, a single wave: the "scanner") reads the
// counts in index order, keeps the running sum, and writes every tile's prefix back; the
// tile then polls its own prefix, one 8-byte load.  Per tile that is one store and a few
// polled loads on lines shared with few other tiles.  (Having every tile read its
// predecessors' counts itself -- a look-back window or a tree -- makes a few hot lines that
// thousands of tiles read at once, and those reads queue up at one memory channel.)
//
// Forward progress does not rest on the order in which workgroups are started.  A workgroup
// publishes its count before it waits for anything, the scanner waits only for counts, and
// a workgroup whose prefix has not come after kPatience polls stops waiting and counts what
// lies before its tile itself, from the call's inputs alone (prefix_from_bitmap,
// prefix_from_input): slow, but then every workgroup that has been started ends, whatever
// the others do, and every workgroup is started in the end.  The scanner's own wait is
// bounded (kSpinLimit): if it runs out the call ends with the error word set.
//
// Entries are value + 1 (0 = not published), written and read with relaxed
// device-scope atomics: the entry is the only thing that is communicated.

// ---- timeline (only in a build with -DBT_TIMELINE) ---------------------------------------------
// Every slot of a bt_compress / bt_decompress launch leaves times of the 100 MHz device
// clock in the caller's buffer (8 words per slot: loads asked for, counted, prefix seen, stores
// issued, -, polls), and the scanner two words per pass that consumed something (time, first
// slot << 32 | end slot), after the slots' words.
#ifdef BT_TIMELINE
__device__ uint64_t *g_timeline = nullptr;
__device__ uint32_t g_timeline_tiles = 0, g_timeline_passes = 0;
// read the recording state once per kernel: a stamp must not cost a memory round trip of its own
#define BT_TL_INIT uint64_t *const tl_buf = g_timeline; const uint32_t tl_tiles = g_timeline_tiles; (void)tl_buf; (void)tl_tiles
#define BT_TL(slot, k)                                                                            \
    do {                                                                                          \
        if (threadIdx.x == 0 && tl_buf != nullptr && (slot) < tl_tiles)                           \
            tl_buf[8 * (size_t)(slot) + (k)] = wall_clock64();                                    \
    } while (0)
#define BT_TL_VALUE(slot, k, v)                                                                   \
    do {                                                                                          \
        if (threadIdx.x == 0 && tl_buf != nullptr && (slot) < tl_tiles)                           \
            tl_buf[8 * (size_t)(slot) + (k)] = (v);                                               \
    } while (0)
#else
#define BT_TL_INIT do {} while (0)
#define BT_TL(slot, k) do {} while (0)
#define BT_TL_VALUE(slot, k, v) do {} while (0)
#endif

__device__ __forceinline__ uint64_t ws_load64(const void *p) {
    return __hip_atomic_load(static_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ws_store64(void *p, uint64_t v) {
    __hip_atomic_store(static_cast<uint64_t *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ws_store32(void *p, uint32_t v) {
    __hip_atomic_store(static_cast<uint32_t *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// nnz, which a host may be looking at while the kernel runs: one store that everybody sees
__device__ __forceinline__ void store_nnz(uint64_t *nnz, const uint64_t v) { __hip_atomic_store(nnz, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
// count + 1 of `tile` in copy c
__device__ __forceinline__ char *ws_count(char *ws, uint32_t tile, uint32_t copy) {
    return ws + kHeaderBytes + (size_t)(tile >> 8) * kBlockBytes + 1024u * copy + 4u * (tile & 255u);
}
// prefix + 1 of `tile` in copy c
__device__ __forceinline__ char *ws_prefix(char *ws, uint32_t tile, uint32_t copy) {
    return ws + kHeaderBytes + (size_t)(tile >> 8) * kBlockBytes + 2048u + 2048u * copy + 8u * (tile & 255u);
}

// The same value in every lane: tell the compiler, so that what is built on it stays in scalar registers.
__device__ __forceinline__ uint32_t uniform32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    return ((uint64_t)uniform32((uint32_t)(v >> 32)) << 32) | uniform32((uint32_t)v);
}

// Polls after which a wait is given up: what the caller asked for in the header, else the
// built-in limit.  Read once, before the wait (a load inside the polling loop would
// lengthen every poll by a round trip).
__device__ __forceinline__ uint32_t wait_limit(const uint32_t *hdr) {
    const uint32_t asked = hdr[kHdrSpinLimit];          // never written by a kernel
    return asked != 0 ? asked : kSpinLimit;
}

// Polls after which a tile's workgroup counts for itself instead of waiting on.  Looked at every 256th poll
// only: read from the header then, it costs neither a register nor a round trip per poll.
__device__ __forceinline__ uint32_t patience_of(const uint32_t *hdr) {
    const uint32_t asked = hdr[kHdrPatience];          // never written by a kernel
    return asked != 0 ? asked : kPatience;
}

// Whether the header's mute word, which is for tests, reaches `level`.  Looked at in the instrumented build only: a look costs
// launches without a scanner 1 to 2 % and batches 0.5 to 1 %.
__device__ __forceinline__ bool told_nothing(const uint32_t *hdr, const uint32_t level) {
#ifdef BT_TIMELINE
    return uniform32(hdr[kHdrMute]) >= level;
#else
    (void)hdr, (void)level;
    return false;
#endif
}

// A call is over as far as the header is concerned (one lane, once every slot's workgroup has published its count and
// hence has read the header): count it, and leave the entries to the next call.
// (A call without a slot, on empty tensors only, has left nothing and cleared nothing.)
// `calls`: its count as it was when this call began, read then: read here it would be waited for, behind every store before it.
__device__ __forceinline__ void header_finish(uint32_t *hdr, const uint32_t n_slots, const uint32_t cur, const uint32_t calls) {
    if (n_slots != 0)
        __hip_atomic_store(&hdr[kHdrEntries], n_slots | ((cur ^ 1u) << 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&hdr[kHdrCalls], calls + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The scanner: one wave.  Workgroups come and go (one per tile) and a count is published as soon as its tile
// has arrived; the scanner takes a few rows of 128 counts starting at the frontier's row in every pass, consumes
// the leading run of published ones (to the slot, not to the row) and asks again.  Every tile of a launch waits
// for the pass that reaches it, so the launch pays for each instruction of this one wave:
//   - what is the same in all lanes (frontier, running sum) is kept in scalar registers;
//   - a lane takes two neighbouring slots (slots 2 i and 2 i + 1 of the row, one 8-byte load), sums its two counts
//     before the DPP prefix sum over the lanes, and stores its two prefixes with one 16-byte store;
//   - a row's prefixes are stored as soon as they are known, and rows behind the first unpublished slot are not
//     looked at.
// The frontier's row is summed again from its first slot in every pass (the slots done before still hold their
// counts, and they are given the prefixes they have already), so the running sum kept between passes is the one
// at that row's start.  The first tile of a batch's tensor marks its count (kFirstTile): where one lies inside a row, the slots
// from there on leave out what was summed before it, which a running maximum over the lanes finds.  All rows are asked for before anything is
// written: on this hardware one counter tracks a wave's loads and stores in order of issue, so a load waited for
// after a store would also wait for that store.  At the end the scanner advances the header for the next call.
// Measured alternatives, all slower or no faster: one slot per lane (rows of 64; 1 to 1.5 % slower), four or
// eight slots per lane (loads and stores spread over more lines), four waves with a window of 28 rows and an
// exchange through LDS, four waves taking rows round robin with the running sum handed on through LDS, a second
// wave that does the stores, whole rows only, a wider window when the last one was used up, more rows per pass
// (restoration is best with two, compression with three).
// A batch's tensors lie slot behind slot.  (They used to start at multiples of 128 slots, with empty slots between, and the sum
// restarted with a row: the 49 tensors of a ResNet-50 at one image took 6,272 slots for 1,200 tiles, and the scanner hands out
// about 220 a microsecond.  Measured, us, before / after, 70 % zeros: compress fp32 at 1 / 4 / 64 images 32.4 / 16.4, 47.4 / 39.6,
// 518 / 509, bf16 at 1 32.2 / 13.1; restore fp32 28.6 / 14.1, 45.9 / 36.8, 574 / 564, bf16 29.5 / 12.0.  With a loop over the tensors of
// a row instead of the running maximum 4 us more at one image; with one sum over all tensors, from which a tile takes its tensor's
// first entry away, 0.5 us less there but 2 % more at 64 images: every tile of a tensor polls that entry.)
typedef uint32_t bt_u32x4 __attribute__((ext_vector_type(4)));
// Two prefix entries in one store that is written through to where every compute unit sees it.  Only for
// entries below 2^32: their upper halves stay the zero they were, so a reader that polls one entry with an
// 8-byte load sees it change in one piece whatever order the four words land in.
__device__ __forceinline__ void ws_store_two_small(void *p, uint32_t first, uint32_t second) {
    const bt_u32x4 v = {first, 0u, second, 0u};
    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}

constexpr uint32_t kFirstTile = 0x80000000u;      // in a count + 1 of a batched call

template <int kRowScan, class Job> __device__ __forceinline__ void scan_counts(char *ws, const Job &job) {
    const uint32_t lane = threadIdx.x & (kWaveSize - 1);
    uint32_t *hdr = reinterpret_cast<uint32_t *>(ws);
    const uint32_t cur = uniform32(hdr[kHdrEntries]) >> 31, calls = uniform32(hdr[kHdrCalls]);
    const uint32_t n_slots = job.slots();
    uint32_t frontier = 0;     // slots [0, frontier) are done
    uint64_t base = 0;         // stored values of the tensor of the frontier's row of 128 slots in its tiles before that row
    uint64_t sum = 0;          // stored values in all tiles before that row (of one tensor: base)
    uint64_t all = 0;          // ... and before the frontier
    constexpr bool kTotalOfEach = Job::kMany && Job::kTotals;
    uint32_t my_start = 0xffffffffu;      // first slot of the lane's tensor
    uint64_t my_sum = 0;                  // stored values in all tiles before it
    if constexpr (kTotalOfEach) {
        if (lane < job.count()) my_start = job.start(lane);
    }
    uint32_t spins = 0;
    const uint32_t limit = uniform32(wait_limit(hdr));
    const bool mute = told_nothing(hdr, 1);
    const bool wide = uniform32(hdr[kHdrWide]) != 0 || mute;      // never written by a kernel
#ifdef BT_TIMELINE
    uint64_t *const timeline = g_timeline;      // read once: a load in the loop would join the scanner's waits
    uint32_t timeline_pass = 0;
#endif
    while (frontier < n_slots) {
        frontier = uniform32(frontier);
        base = uniform64(base);
        if (Job::kMany) sum = uniform64(sum);
        const uint32_t row = frontier >> 7;
        uint32_t ca[kRowScan], cb[kRowScan];          // count + 1 of the lane's two slots; 0: not published yet, or past the end
#pragma unroll
        for (int j = 0; j < kRowScan; ++j) {
            const uint32_t t = 128u * (row + j) + 2u * lane;
            uint64_t two = 0;
            if (t < n_slots)
                two = __hip_atomic_load(reinterpret_cast<const uint64_t *>(ws_count(ws, t, cur)), __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
            ca[j] = (uint32_t)two;
            cb[j] = t + 1 < n_slots ? (uint32_t)(two >> 32) : 0u;
        }
        const bool small = !wide && (base >> 32) == 0 && (uint32_t)base < 0xF0000000u;   // all of this pass's entries below 2^32
        bool open = true;
        uint32_t new_frontier = frontier;
#pragma unroll
        for (int j = 0; j < kRowScan; ++j) {
            if (open) {
                const uint32_t slot0 = 128u * (row + j);
                const uint64_t bad_a = __ballot(ca[j] == 0), bad_b = __ballot(cb[j] == 0);
                const uint32_t run_a = bad_a == 0 ? 64u : (uint32_t)__builtin_ctzll(bad_a);
                const uint32_t run_b = bad_b == 0 ? 64u : (uint32_t)__builtin_ctzll(bad_b);
                const uint32_t run = uniform32(min(2u * run_a, 2u * run_b + 1u));   // usable slots of the row, in slot order
                const uint32_t row_end = slot0 + run;
                if (row_end > new_frontier) {
                    const bool use_a = 2u * lane < run, use_b = 2u * lane + 1u < run;
                    constexpr uint32_t kValue = Job::kMany ? ~kFirstTile : ~0u;
                    const uint32_t va = use_a ? (ca[j] & kValue) - 1u : 0u, vb = use_b ? (cb[j] & kValue) - 1u : 0u;
                    const uint32_t incl = wave_inclusive_sum(va + vb);
                    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                    char *const entry = ws_prefix(ws, slot0 + 2u * lane, cur);
                    const uint32_t before = incl - va - vb;      // in the row
                    // the lane's two entries, from what the row's sums are counted from
                    const auto store = [&](const uint64_t from_a, const uint64_t from_b) __attribute__((always_inline)) {
                        if (small) {
                            const uint32_t pa = (uint32_t)from_a + before, pb = (uint32_t)from_b + before + va;
                            if (use_b) ws_store_two_small(entry, pa, pb);
                            else if (use_a) ws_store32(entry, pa);
                        } else {
                            if (use_a && !mute) ws_store64(entry, from_a + before);
                            if (use_b && !mute) ws_store64(entry + 8, from_b + before + va);
                        }
                    };
                    new_frontier = row_end;
                    uint64_t row_base = base;
                    const bool first_a = Job::kMany && use_a && ca[j] >= kFirstTile, first_b = Job::kMany && use_b && cb[j] >= kFirstTile;
                    if (!Job::kMany || __ballot(first_a || first_b) == 0) {
                        store(base + 1, base + 1);
                    } else {
                        // one more than what the row's tensor so far has in the row, at the slots where a tensor begins;
                        // sums only grow, so the last of these is the largest
                        const uint32_t at_a = first_a ? before + 1u : 0u, at_b = first_b ? before + va + 1u : 0u;
                        const uint32_t last = wave_inclusive_max(max(at_a, at_b));
                        const uint32_t skip_a = max(at_a, BT_DPP(0, last, 0x138, 0xf, true));      // wave_shr:1
                        const uint32_t skip_b = max(at_b, skip_a);
                        store(skip_a != 0 ? 2 - (uint64_t)skip_a : base + 1, skip_b != 0 ? 2 - (uint64_t)skip_b : base + 1);
                        row_base = 1 - (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)last, 63);
                        if constexpr (kTotalOfEach) {
                            const uint32_t at = my_start - slot0;
                            const int from = (int)(4u * (at >> 1));      // (not looked at where the lane's tensor begins elsewhere)
                            const uint32_t sums = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)before);
                            const uint32_t first = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)va);
                            if (at < run) my_sum = sum + sums + ((at & 1u) != 0 ? first : 0u);
                        }
                    }
                    all = uniform64((Job::kMany ? sum : base) + total);
                    if (run == 128u) {
                        base = uniform64(row_base + total);
                        sum = all;
                    }
                }
                open = run == 128u;
            }
        }
        // the scanner's wait for the call's counts is bounded in passes, fruitful or not
        if (++spins > limit) {
            if (lane == 0) __hip_atomic_store(&hdr[kHdrError], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        if (new_frontier == frontier) {
            __builtin_amdgcn_s_sleep(kScannerSleep);
            continue;
        }
#ifdef BT_TIMELINE
        if (timeline != nullptr && lane == 0 && timeline_pass < g_timeline_passes) {
            timeline[8 * (size_t)g_timeline_tiles + 2 * timeline_pass] = wall_clock64();
            timeline[8 * (size_t)g_timeline_tiles + 2 * timeline_pass + 1] = ((uint64_t)frontier << 32) | new_frontier;
            ++timeline_pass;
        }
#endif
        frontier = new_frontier;
    }
    if constexpr (kTotalOfEach) {
        static_assert(kMaxBatchCompress < kWaveSize, "a lane per tensor and one behind the last");
        if (my_start >= n_slots) my_sum = all;      // (empty tensors at the end, and the lane behind the last tensor)
        const uint64_t next = __shfl_down((unsigned long long)my_sum, 1, kWaveSize);
        if (lane < job.count()) store_nnz(job.nnz(lane), next - my_sum);
    } else if constexpr (Job::kTotals) {
        if (lane == 0) store_nnz(job.nnz(0), all);
    }
    if (lane == 0) {
        // every slot's workgroup has published its count by now, hence has read the header: advance it
        header_finish(hdr, n_slots, cur, calls);
    }
}

// What a workgroup reads from the header before it publishes anything (in compression once its tile's loads are on their
// way).  The header is rewritten once every slot of the call has published, so no wave may read it after any wave of its
// workgroup has published a count.
// A workspace on which a wait was given up is in no defined state: later calls on it do nothing (and stay away from its
// stale entries) until bt_workspace_init has been run.  The error word may be set while a workgroup's waves read
// it, so a wave that sees it tells the others where their totals meet (kWaveFailed) and they leave together.
struct Epoch {
    uint32_t cur;          // copy of the entries this call uses
    uint32_t prev_slots;   // entries the previous call used in the other copy
    uint32_t calls;
    bool failed;
};
constexpr uint32_t kWaveFailed = 0xffffffffu;      // (no wave's total)

struct HeaderWords { uint32_t entries, error, calls; };      // as they come from memory
__device__ __forceinline__ HeaderWords read_header(const char *ws) {
    const uint32_t *hdr = reinterpret_cast<const uint32_t *>(ws);
    return HeaderWords{hdr[kHdrEntries], hdr[kHdrError], hdr[kHdrCalls]};
}
__device__ __forceinline__ Epoch epoch_of(const HeaderWords h) {
    const uint32_t entries = uniform32(h.entries);
    return Epoch{entries >> 31, entries & 0x7fffffffu, uniform32(h.calls), uniform32(h.error) != 0};
}

template <int W> __device__ __forceinline__ bool any_wave_failed(const uint32_t (&totals)[W]) {
    bool any = false;
#pragma unroll
    for (int w = 0; w < W; ++w) any = any || uniform32(totals[w]) == kWaveFailed;
    return any;
}

// Compression of a small tensor (see compress_common) has no scanner: a tile's first wave reads the counts of all tiles
// before it itself, which leaves two of the four hops through memory (count store -> scanner load -> prefix store ->
// tile poll).  The last tile's workgroup, which needs every count, does what the scanner does at the end: nnz and the header.
// (With thousands of tiles the same few lines would be polled by all of them at once.)
constexpr uint32_t kDirectSlots = 256;
static_assert(kDirectSlots % 128 == 0, "a lane takes two neighbouring slots of each 128");
constexpr uint32_t kLog2Xcds = 3;         // consecutive workgroups go to the eight XCDs in turn
// Up to kQuarterSlots tiles all four waves of a tile read the counts, a quarter of the slots each (wait_for_quarter): one wave's
// load of 128 counts and the registers for it, four times in a row, would cost more than the scanner's two hops.
constexpr uint32_t kQuarterSlots = 512;
static_assert(kQuarterSlots == 128 * kWaves, "two neighbouring slots a lane");

// The number of values before `slot`, summed from the published counts by one wave, or false if they are not all there.
__device__ __forceinline__ bool sum_counts(char *ws, const uint32_t slot, const uint32_t cur, uint64_t &sum) {
    constexpr int kSteps = kDirectSlots / 128;      // of two neighbouring slots a lane
    uint64_t two[kSteps];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const uint32_t at = 128u * i + 2u * (uint32_t)lane_number();
        two[i] = 0;
        if (at < slot) two[i] = ws_load64(ws_count(ws, at, cur));
    }
    bool missing = false;
    uint32_t mine = 0;
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const uint32_t at = 128u * i + 2u * (uint32_t)lane_number();
        const uint32_t ca = (uint32_t)two[i], cb = (uint32_t)(two[i] >> 32);
        missing = missing || (at < slot && ca == 0) || (at + 1 < slot && cb == 0);
        mine += (at < slot ? ca - 1u : 0u) + (at + 1 < slot ? cb - 1u : 0u);
    }
    if (__ballot(missing) != 0) return false;
    sum = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(mine), 63);
    return true;
}

// Pause between two polls of a tile for its prefix.  A launch that the GPU swallows in one go wants the answer soon; where
// thousands of workgroups come and go, the polls of the two thousand resident ones stand in the way of the scanner's
// and of the values'.  Measured with pauses of 4 / 16 / 32 x 64 clocks, us: fp32 at 50 % zeros, restore 4.5 M elements (549
// tiles) 8.5 / 8.7 / 8.9, 8 M 11.4 / 11.6 / 12.0, 12.8 M (1563) 16.3 / 16.2 / 16.5, 25.7 M (3136) 26.9 / 26.7 / 27.0; compress 4 M (489)
// 8.5 / 8.7 / 8.9, 8 M 11.2 / 11.3 / 11.4, 25.7 M 28.4 / 28.2 / 29.1; restore fp64 2.1 M (513) 8.1 / 8.5 / 8.5, fp16 206 M (12,544 tiles, 5 % zeros)
// 141.4 / 141.3 / 141.2; the 49 tensors of a ResNet-50 (75,068 slots) restore 611 / 603 / 570, compress 530 / 519 / 515.
__device__ __forceinline__ void poll_pause(const uint32_t n_slots) {
    if (n_slots >= 8192) __builtin_amdgcn_s_sleep(32);
    else if (n_slots > 1536) __builtin_amdgcn_s_sleep(16);
    else __builtin_amdgcn_s_sleep(4);
}

// The wait of a tile's first wave for the scanner: the number of values before its slot.  `itself` counts what precedes the
// tile from the call's input, for a wave that stops waiting.
template <class Itself>
__device__ __forceinline__ uint64_t wait_for_prefix(char *ws, const uint32_t slot, const uint32_t n_slots, const uint32_t cur, uint32_t &polls,
                                                    const Itself &itself) {
    for (;;) {
        const uint64_t v = uniform64(ws_load64(ws_prefix(ws, slot, cur)));
        ++polls;
        if (v != 0) return v - 1;
        if (__builtin_expect((polls & 255u) == 0 && polls > patience_of(reinterpret_cast<const uint32_t *>(ws)), 0)) return itself();
        poll_pause(n_slots);
    }
}

// The same in a launch without a scanner.  `complete`: this is the last tile, and it has seen every count.
template <class Itself>
__device__ __forceinline__ uint64_t wait_for_counts(char *ws, const uint32_t slot, const uint32_t n_slots, const uint32_t cur, uint32_t &polls, bool &complete,
                                                    const Itself &itself) {
    uint32_t *const hdr = reinterpret_cast<uint32_t *>(ws);
    const bool last = slot + 1 == n_slots;
    const bool deaf = told_nothing(hdr, last ? 2 : 1);
    uint64_t v = 0;
    complete = false;
    while (deaf || !sum_counts(ws, slot, cur, v)) {
        ++polls;
        if (!last && (polls & 255u) == 0 && polls > patience_of(hdr)) return itself();
        if (last && polls >= wait_limit(hdr)) {      // its wait is bounded like the scanner's
            if (lane_number() == 0) __hip_atomic_store(&hdr[kHdrError], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return itself();
        }
        __builtin_amdgcn_s_sleep(kScannerSleep);
    }
    complete = last;
    return v;
}

// A wave's share of the wait in a launch of up to kQuarterSlots tiles: the number of values in the tiles before `slot` among the
// wave's quarter of the slots, or kWaveFailed if the counts have not all been there for too many polls.  The last tile's wait is bounded
// like the scanner's, fruitful or not: a limit of one poll makes every such call fail.
__device__ __forceinline__ uint32_t wait_for_quarter(char *ws, const uint32_t slot, const bool last, const uint32_t cur, const int wave, uint32_t &polls) {
    uint32_t *const hdr = reinterpret_cast<uint32_t *>(ws);
    const bool deaf = told_nothing(hdr, last ? 2 : 1);
    uint32_t limit = 0;
    if (last) limit = uniform32(wait_limit(hdr));
    for (;;) {
        const uint32_t at = 128u * (uint32_t)wave + 2u * (uint32_t)lane_number();
        uint64_t two = 0;
        if (at < slot) two = ws_load64(ws_count(ws, at, cur));
        const uint32_t ca = at < slot ? (uint32_t)two : 1u, cb = at + 1 < slot ? (uint32_t)(two >> 32) : 1u;
        ++polls;
        if (last && polls >= limit) return kWaveFailed;
        if (__ballot(deaf || ca == 0 || cb == 0) == 0) return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(ca + cb - 2u), 63);
        if (!last && (polls & 255u) == 0 && polls > patience_of(hdr)) return kWaveFailed;
        __builtin_amdgcn_s_sleep(kScannerSleep);
    }
}

// What the four waves have found, added up.  If one has given up, every wave counts what precedes the tile from the call's input
// (`itself`), and the call has failed if this is the last tile, which was to end it.
template <class Itself>
__device__ __forceinline__ uint64_t add_quarters(char *ws, const uint32_t (&found)[kWaves], const bool last, bool &complete, const Itself &itself) {
    uint32_t sum = 0;
    bool gave_up = false;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t q = uniform32(found[w]);
        gave_up = gave_up || q == kWaveFailed;
        sum += q;
    }
    complete = last && !gave_up;
    if (__builtin_expect(!gave_up, 1)) return sum;
    if (last && threadIdx.x == 0) __hip_atomic_store(&reinterpret_cast<uint32_t *>(ws)[kHdrError], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return itself();
}

// Zero what the previous call left in the other copy of the workspace entries: the blocks of slots
// [0, prev_slots), shared out over this call's `workers` workgroups; a thread takes one slot of a block.
__device__ __forceinline__ void zero_previous(char *ws, const Epoch ep, const uint32_t worker, const uint32_t workers) {
    static_assert(kBlock == kSlotsPerBlock, "a thread per slot of a block");
    const uint32_t other = ep.cur ^ 1u;
    for (uint64_t b = worker; b * kSlotsPerBlock < ep.prev_slots; b += workers) {
        char *const entries = ws + kHeaderBytes + b * kBlockBytes;
        // (written out, with the uniform part of the addresses in scalar registers: this runs where vector registers are short)
        asm volatile("global_store_dword %0, %1, %2 sc1" : : "v"(4u * threadIdx.x), "v"(0u), "s"(entries + 1024u * other) : "memory");
        asm volatile("global_store_dwordx2 %0, %1, %2 sc1" : : "v"(8u * threadIdx.x), "v"((uint64_t)0), "s"(entries + 2048u + 2048u * other) : "memory");
    }
}

// A lane's E-bit non-zero masks of all rows, packed RPM rows to a register.
#define BT_MASK(S_, mp, k) (((mp)[(k) / Geo<S_>::RPM] >> (Geo<S_>::E * ((k) % Geo<S_>::RPM))) & ((1u << Geo<S_>::E) - 1u))

// Per-row popcounts -> exclusive rank of each lane inside its row (two rows per
// register, 16-bit fields: a row holds at most 512 non-zeros) and the row totals
// (same packing, wave-uniform).
template <int S, int R>
__device__ __forceinline__ void rank_rows(const uint32_t (&mp)[Geo<S, R>::MW], uint32_t (&rank2)[R / 2],
                                          uint32_t (&total2)[R / 2]) {
#pragma unroll
    for (int k = 0; k < R; k += 2) {
        const uint32_t packed = (uint32_t)__popc(BT_MASK(S, mp, k)) | ((uint32_t)__popc(BT_MASK(S, mp, k + 1)) << 16);
        const uint32_t incl = wave_inclusive_sum(packed);
        rank2[k / 2] = incl - packed;
        total2[k / 2] = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
}
#define BT_FIELD(arr2, k) (((arr2)[(k) / 2] >> (16 * ((k) & 1))) & 0xffffu)

// ---- Algorithm 1: dense -> bitmap -------------------------------------------------------

// 16 bytes of LDS at an element-aligned byte offset.  The misalignment is the same in all lanes (it is that of the
// workgroup's place in the value array).
template <int S> __device__ __forceinline__ uint4 lds_load_shifted(const unsigned char *p, const bool odd_half) {
    typedef uint32_t dword4 __attribute__((ext_vector_type(4), aligned(4)));
    if (S == 2 && odd_half) {
        const uint32_t *q = reinterpret_cast<const uint32_t *>(p - 2);
        const dword4 v = *reinterpret_cast<const dword4 *>(q);
        const uint32_t next = q[4];
        return make_uint4(__builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16),
                          __builtin_amdgcn_alignbit(v.w, v.z, 16), __builtin_amdgcn_alignbit(next, v.w, 16));
    }
    const dword4 v = *reinterpret_cast<const dword4 *>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Write `cnt` elements to gdst with aligned 16-byte stores of kThreads threads (`t`: this one's number).  kPlaced: they
// lie in LDS from element `pad` of `run` on, pad being gdst's distance from the 16-byte boundary before it.  Otherwise
// they lie from the start of `run` on, as they do when they are compacted before the prefix tells what gdst is, and
// LDS is read at the shift that lines up with gdst.  The first and
// the last vector go element by element, so nothing outside [gdst, gdst + cnt) is touched.  All LDS reads of the inner
// vectors are issued before the first store and the two edge vectors are left to 2 E threads at the end: this runs
// after the tile has received its prefix, where every instruction delays the tile's exit.
template <int S, int kThreads, int kMaxBytes, bool kPlaced>
__device__ __forceinline__ void run_store(const unsigned char *run, char *gdst, const uint32_t cnt, const int t) {
    constexpr int E = Geo<S>::E;
    constexpr int kSteps = (kMaxBytes / kVecBytes + kThreads - 1) / kThreads;      // inner vectors a thread (at most kMaxBytes / 16 - 1 in all)
    if (cnt == 0) return;
    const uint32_t pad = (uint32_t)(reinterpret_cast<uintptr_t>(gdst) & (kVecBytes - 1)) / S;   // elements
    char *const gvec = gdst - (size_t)pad * S;  // 16-byte aligned; may start before gdst
    const uint32_t hi_valid = pad + cnt;
    const uint32_t n_vec = (hi_valid + E - 1) / E;
    const uint32_t shift = kPlaced ? 0u : pad;
    const bool odd_half = S == 2 && (shift & 1u) != 0;
    uint4 x[kSteps];
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const uint32_t v = 1u + (uint32_t)t + (uint32_t)kThreads * i;
        if (v + 1 < n_vec)
            x[i] = kPlaced ? *reinterpret_cast<const uint4 *>(run + (size_t)v * kVecBytes) : lds_load_shifted<S>(run + (v * E - shift) * S, odd_half);
    }
#pragma unroll
    for (int i = 0; i < kSteps; ++i) {
        const uint32_t v = 1u + (uint32_t)t + (uint32_t)kThreads * i;
        if (v + 1 < n_vec) stream_store<kCompressNtStore>(reinterpret_cast<uint4 *>(gvec + (size_t)v * kVecBytes), x[i]);
    }
    // the first and the last vector, an element a thread: thread j < E element j of the first, thread E + j element j
    // of the last, each only if it lies inside [pad, pad + cnt)
    if (t < 2 * E) {
        const uint32_t e = t < E ? (uint32_t)t : (n_vec - 1) * E + (uint32_t)(t - E);
        if (e >= pad && e < hi_valid && (t < E || n_vec > 1)) {
            if (S == 8) reinterpret_cast<uint64_t *>(gvec)[e] = reinterpret_cast<const uint64_t *>(run)[e - shift];
            else if (S == 4) reinterpret_cast<uint32_t *>(gvec)[e] = reinterpret_cast<const uint32_t *>(run)[e - shift];
            else reinterpret_cast<uint16_t *>(gvec)[e] = reinterpret_cast<const uint16_t *>(run)[e - shift];
        }
    }
}

// Put the kept elements of one row of a wave into LDS: lane by lane from byte `rb` before `dump` on, in element order.
// Every element is written, a dropped one to `dump`, a place nobody reads: a select on the address instead of
// a branch around the write keeps the execution mask alone.
template <int S> __device__ __forceinline__ void scatter_row(unsigned char *const dump, int rb, const uint32_t mk, const uint4 x) {
    const uint32_t d[4] = {x.x, x.y, x.z, x.w};
    if (S == 8) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int keep = (int)((mk >> j) & 1u);
            *reinterpret_cast<bt_u2 *>(dump + __mul24(keep, rb)) = bt_u2{d[2 * j], d[2 * j + 1]};
            rb += keep * S;
        }
    } else if (S == 4) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int keep = (int)((mk >> j) & 1u);
            *reinterpret_cast<uint32_t *>(dump + __mul24(keep, rb)) = d[j];
            rb += keep * S;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int keep = (int)((mk >> j) & 1u);
            *reinterpret_cast<uint16_t *>(dump + __mul24(keep, rb)) = (uint16_t)(d[j >> 1] >> (16 * (j & 1)));
            rb += keep * S;
        }
    }
}

// What a compressing workgroup does when the scanner's answer for its tile does not come: its first
// wave counts the kept elements of the tensor before the tile itself, with the same test.  Slow (the
// whole input up to the tile), but it needs nothing from any other workgroup.
template <int S, int R, int KEEP>
__device__ __forceinline__ uint64_t prefix_from_input(const void *__restrict__ in, const uint32_t tile, const float threshold_f,
                                                   const double threshold, const int lane) {
    const uint64_t vectors = (uint64_t)tile * (Geo<S, R>::TILE / Geo<S, R>::E);      // all of them whole and inside the tensor
    const uint4 *const end = static_cast<const uint4 *>(in) + vectors;
    uint32_t share = 0;      // at most BT_MAX_ELEMENTS / 64
#pragma unroll 1
    for (const uint4 *q = static_cast<const uint4 *>(in) + lane; q < end; q += kWaveSize)
        share += (uint32_t)__popc(keep_mask<S, KEEP>(*q, threshold_f, threshold));
    return wave_total_of(share);
}

// bt_compress and its relatives (pruning, dense output, tile index, batches).  Tiles of R rows a lane; with DIRECT = 0
// workgroup 0 is the scanner (one wave of it) and workgroup 1 + t compresses slot t, otherwise (launches on one tensor of up to
// DIRECT tiles, see compress_common) workgroup t does and sums the counts before its tile itself.
// 1. load: lane l of row k owns elements wave_e0 + k * ROW + l * E ... + E - 1 of its wave's quarter of the
//    tile; all R rows are asked for at once.
// 2. the test of Algorithm 1 (on the bit pattern), or the pruning test; masks packed RPM rows to a register;
//    ranks by one DPP wave prefix sum per two rows.
// 3. bitmap words: G lanes OR their E-bit masks into one 32-bit word.
// 4. the waves' totals meet in LDS and the tile's count is published.  While the prefix is on its way the kept elements
//    are compacted in LDS at their ranks (all of them if the tile's values fit, as they do up to 62 % non-zero elements of
//    eight rows and always of fewer; else each wave's first rows) and the waves that do not poll store their bitmap words;
//    then the first wave polls.
// 5. values: with the prefix known, the compacted run is read back at the shift that lines it up with a 16-byte boundary
//    of the value array and written with aligned stores, by the whole workgroup; a tile that did not fit goes
//    PHASE rows at a time, each wave its own.
// What bounds it: the memory system on large tensors (fp32, 205 M elements: 6.2 TB/s), the chain load, count, scan,
// prefix, store on ordinary ones, so what follows the prefix is kept short.  Compacting before the wait instead of
// after it measured, us: configuration 2 (fp32, 25.7 M elements, 50 % zeros) 30.7 -> 29.5, at 90 % zeros 26.5 -> 24.9;
// bf16 67 M elements at 65 % zeros 37.1 -> 35.2; fp16 206 M elements at 95 % zeros 88.9 -> 83.0, at 5 % 138.1 (does not fit)
// -> 138.1; fp64 25.7 M 54.9 -> 53.4; the 49 tensors of a ResNet-50 539 -> 524; activation call fp32 5.5 M 13.4 -> 11.5 (10.6 since
// it keeps nothing in scratch).  No kernel may: a value that comes back from scratch behind the stores waits for them.
// The staging area is what eight workgroups leave each other of a compute unit's 160 KiB: more would cost occupancy.
// The workgroup ends with its stores on their way: nothing waits for them to land.  (A persistent version
// of this kernel -- as many workgroups as are resident, each taking tiles w, w + G, ..., the next tile's loads
// asked for before the current tile's prefix wait, compacted values parked in rings in LDS -- was built and
// measured: 1 % faster on a 25.7 M element fp32 tensor, 5 to 15 % slower on 16-bit and on larger tensors.)
template <int S, int R, int DIRECT, int KEEP, bool DENSE, class Job>
__global__ __launch_bounds__(kBlock, kCompressOcc) void compress_kernel(const Job job, char *ws, const double threshold, const float threshold_f) {
    using G = Geo<S, R>;
    constexpr int E = G::E;
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[G::STAGE + kVecBytes];
    __shared__ uint64_t s_tile_prefix;
    __shared__ uint32_t s_wave_total[kWaves], s_found[kWaves];
    constexpr bool kQuarters = DIRECT > (int)kDirectSlots;
    // (of the launches of few tiles of two rows one workgroup in eight works, see kOneXcdSlots)
    constexpr bool kMayBeApart = R == 2 && !DENSE;
    const uint32_t n_slots = kMayBeApart ? job.slots() : gridDim.x - (DIRECT ? 0u : 1u);
    const uint32_t apart = kMayBeApart && gridDim.x != n_slots ? kLog2Xcds : 0u;
    if (kMayBeApart && (blockIdx.x & ((1u << apart) - 1u)) != 0) return;
    if (!DIRECT && blockIdx.x == 0) {
        if (threadIdx.x < kWaveSize && !epoch_of(read_header(ws)).failed) scan_counts<3>(ws, job);
        return;
    }
    BT_TL_INIT;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it in a scalar register
    const uint32_t slot = kMayBeApart ? blockIdx.x >> apart : blockIdx.x - (DIRECT ? 0u : 1u);
    const Slot sl = job.at(slot);
    const uint32_t tile = sl.tile;
    const uint64_t n = job.n(sl.item);
    const void *const in = job.in(sl.item);
    const uint64_t n_words = (n + 31) >> 5;
    const uint64_t wave_e0 = (uint64_t)tile * G::TILE + (uint64_t)wave * G::WAVE;
    const bool full = (uint64_t)(tile + 1) * G::TILE <= n;

    // (1), (2)
    uint4 x[R];
    uint32_t mp[G::MW], rank2[R / 2], total2[R / 2];
#pragma unroll
    for (int i = 0; i < G::MW; ++i) mp[i] = 0;
    BT_TL(slot, 0);
    if (__builtin_expect(full, 1)) {
        const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const char *>(in) + wave_e0 * S) + lane;
#pragma unroll
        for (int k = 0; k < R; ++k) x[k] = stream_load<kCompressNtLoad>(p + k * kWaveSize);
    }
    // The header is looked at while the tile is on its way (the tile's loads stay before it).
    asm volatile("" ::: "memory");
    // written at the end of the previous call; constant until every slot of this call has published
    const HeaderWords header = read_header(ws);
    if (full) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            uint32_t mk = keep_mask<S, KEEP>(x[k], threshold_f, threshold);
            asm volatile("" : "+v"(mk));             // row k has arrived: its mask exists from here on
            mp[k / G::RPM] |= mk << (E * (k % G::RPM));
        }
    } else {
        // A tensor's ragged last tile: what is there of it in whole vectors, all rows at once, then the elements of the
        // vector in which the tensor ends.  Elements beyond n are 0, which no test keeps.  (Row after row, element by element, the
        // tile had its values a microsecond or two after the others, with every tensor whose size is no multiple of a tile.
        // Together with store_vec_guarded's early return, us: bf16 5.9 M elements compress 9.3 -> 8.3, activation call 12.3 -> 9.6, 320 k 4.9 ->
        // 4.5 and 6.4 -> 5.5; fp32 160 k 4.6 -> 4.3 and 5.3 -> 4.7; the 49 tensors of a ResNet-50 at one image, bf16, 13.2 -> 10.9.)
        const uint32_t left = n <= wave_e0 ? 0u : n - wave_e0 < (uint64_t)G::WAVE ? (uint32_t)(n - wave_e0) : (uint32_t)G::WAVE;      // elements of this wave
        const char *const quarter = static_cast<const char *>(in) + wave_e0 * S;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const uint32_t at = (uint32_t)(k * G::ROW + lane * E);
            x[k] = make_uint4(0, 0, 0, 0);
            if (at + E <= left) x[k] = stream_load<kCompressNtLoad>(reinterpret_cast<const uint4 *>(quarter + at * S));
        }
        const uint32_t whole = left / E * E;
        if (whole != left) {
            const uint4 v = load_vec_guarded<S>(in, wave_e0 + whole, n);
            const uint32_t d[4] = {uniform32(v.x), uniform32(v.y), uniform32(v.z), uniform32(v.w)};
#pragma unroll
            for (int k = 0; k < R; ++k) {
                if ((uint32_t)(k * G::ROW + lane * E) == whole) x[k] = make_uint4(d[0], d[1], d[2], d[3]);
            }
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            // (A loop of its own: where both kinds of tile meet before it, the wait for row 0 becomes one for all rows.  And nothing of
            // a row's test before its turn: halves widened ahead take registers there are not.)
            asm volatile("" : "+v"(x[k].x), "+v"(x[k].y), "+v"(x[k].z), "+v"(x[k].w));
            uint32_t mk = keep_mask<S, KEEP>(x[k], threshold_f, threshold);
            asm volatile("" : "+v"(mk));
            mp[k / G::RPM] |= mk << (E * (k % G::RPM));
        }
    }
    // Keep the masks as values of their own: otherwise the compiler keeps one compare
    // result (a scalar register pair) per element alive until the values are written.
#pragma unroll
    for (int i = 0; i < G::MW; ++i) asm volatile("" : "+v"(mp[i]));
    rank_rows<S, R>(mp, rank2, total2);
    uint32_t wave_total = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) wave_total += BT_FIELD(total2, k);

    // (3) lane (g * G + i) keeps the word of row r0 + i, group g: one store per G rows.
    constexpr int kWordRegs = (R + G::G - 1) / G::G;
    uint32_t word[kWordRegs];
    {
        const int i = lane % G::G;
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += G::G) {
            word[r0 / G::G] = 0;
#pragma unroll
            for (int k = r0; k < r0 + G::G && k < R; ++k) {
                const uint32_t w = group_or<G::G>(BT_MASK(S, mp, k) << (uint32_t)(E * i));
                if (i == k - r0) word[r0 / G::G] = w;
                // finish this row's word now: left alone, the compiler sinks the selects below
                // the compaction in (4) and keeps one partial result per row alive across it
                asm volatile("" : "+v"(word[r0 / G::G]));
            }
        }
    }

    const auto store_words = [&]() {
        uint32_t *const bitmap = job.bitmap(sl.item);
        const int g = lane / G::G, i = lane % G::G;
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += G::G) {
            const uint64_t widx = (wave_e0 >> 5) + (uint64_t)(r0 + i) * G::WPR + (uint64_t)g;
            if (r0 + i < R && widx < n_words) bitmap[widx] = word[r0 / G::G];
        }
    };
    // (4)
    const Epoch ep = epoch_of(header);
    if (lane == 0) s_wave_total[wave] = ep.failed ? kWaveFailed : wave_total;
    lds_barrier();                      // also: every wave has read the header before the first wave publishes anything
    if (any_wave_failed(s_wave_total)) return;
    uint32_t before_wave = 0, tile_total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_wave_total[w];
        if (w < wave) before_wave += c;
        tile_total += c;
    }
    before_wave = uniform32(before_wave);       // the same in every lane: tell the compiler, so that addresses built on it stay scalar
    tile_total = uniform32(tile_total);
    if (tid == 0) ws_store32(ws_count(ws, slot, ep.cur), (tile_total + 1) | (Job::kMany && tile == 0 ? kFirstTile : 0u));
    BT_TL(slot, 1);
    zero_previous(ws, ep, slot, n_slots);

    // What needs no prefix is done while it is on its way.
    // The dense tensor after pruning, if asked for (bt_activation_compress): what survives keeps its bits, the
    // rest is +0.  The dense output may be the input itself (every lane rewrites exactly the vectors it has read).
    const auto store_dense = [&]() __attribute__((always_inline)) {
        void *const dense = job.dense(sl.item);
#pragma unroll
        for (int k = 0; k < R; ++k) {
            uint32_t mk = BT_MASK(S, mp, k);
            if (S == 2 && !DIRECT) asm volatile("" : "+v"(mk));      // (a row's work starts here, as in the compaction below)
            // Masks by arithmetic (0 - bit is all ones or zero), not by compares: see nonzero_mask.  In place, and with the row's
            // address in scalar registers, because vector registers are short: of a dropped element nothing is looked at any
            // more.  (A row's masked copy put 8 to 9 registers of the eight-row kernels into scratch: fp64 5 M elements 18.7 us,
            // now 15.2, 103 M 347 / 340; fp32 12 M 19.8 / 18.1.)
            uint32_t *const d[4] = {&x[k].x, &x[k].y, &x[k].z, &x[k].w};
            if (S == 8) {
#pragma unroll
                for (int j = 0; j < 4; ++j) *d[j] &= 0u - ((mk >> (j >> 1)) & 1u);
            } else if (S == 4) {
#pragma unroll
                for (int j = 0; j < 4; ++j) *d[j] &= 0u - ((mk >> j) & 1u);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *d[j] &= (((mk >> (2 * j)) & 1u) * 0x0000ffffu) | (((mk >> (2 * j + 1)) & 1u) * 0xffff0000u);
            }
            const uint64_t row_e0 = wave_e0 + (uint64_t)k * G::ROW;
            if (full) stream_store<kCompressNtStore>(reinterpret_cast<uint4 *>(static_cast<char *>(dense) + row_e0 * S) + lane, x[k]);
            else store_vec_guarded<S>(dense, row_e0 + (uint64_t)(lane * E), n, x[k]);
        }
    };
    // Before the wait or after it?  Before (but behind the compaction, which has the values in registers too), the stores use
    // memory that would idle while the prefixes of a small launch are on their way, but the polling wave waits for its own
    // first; in a launch that keeps the memory busy they only hold up everybody's polls and values.  Measured, before / after, us,
    // pre-activations without zeros and with half zeros: fp32 6.5 M elements (794 tiles) 12.4 / 13.2 and 12.1 / 12.6, 8 M (977)
    // 14.4 / 14.8 and 13.9 / 13.4, 9 M (1099) 18.3 / 16.3 and 17.4 / 14.8; fp64 3.7 M (904) 13.1 / 13.7 and 12.9 / 12.5, 4.5 M (1099)
    // 18.3 / 15.8 and 17.4 / 14.3; bf16 18 M (1099) 18.3 / 18.9 and 17.4 / 17.7, 20 M (1221) 19.0 / 19.5 and 17.9 / 18.0.
    const bool dense_early = DENSE && n_slots <= kDenseEarlySlots<S>;
    // The bitmap words; the wave that polls keeps its own until afterwards, because a store in flight delays the polling
    // loads, which share its completion counter.  (For 16-bit elements in tiles of eight rows it has no register to keep them in.)
    const bool words_early = (S == 2 && R == kRows) || dense_early || (!kQuarters && wave != 0);
    if (words_early) store_words();

    // The values: if the tile's fit LDS together (62 % of its elements: most activations), all of them are compacted into
    // one run now; if not, each wave's first PHASE rows into a strip of its own.
    constexpr bool kAlwaysStaged = G::STAGE == G::TILE * S;
    const bool staged = kAlwaysStaged || tile_total * S <= (uint32_t)G::STAGE;
    constexpr int kStrip = G::PHASE * G::ROW * S + kVecBytes;      // the rows, and the shift to a 16-byte boundary
    static_assert(kAlwaysStaged || kWaves * kStrip <= G::STAGE, "the waves' strips share the staging area");
    const int run0 = staged ? (int)(before_wave * S) : wave * kStrip;      // byte offset of this wave's first value
    uint32_t row_start = 0;                                                // kept elements of the wave in the rows before
    const auto scatter = [&](const int k, const int from) __attribute__((always_inline)) {
        // byte offset of this lane's next kept element from the spare vector (negative: the values lie before it)
        const int rb = from + (int)((row_start + BT_FIELD(rank2, k)) * S) - G::STAGE;
        uint32_t mk = BT_MASK(S, mp, k);
        asm volatile("" : "+v"(mk));      // (a row's work starts here: nothing of it is done ahead, registers are short)
        scatter_row<S>(s_stage + G::STAGE, rb, mk, make_uint4(x[k].x, x[k].y, x[k].z, x[k].w));
        row_start += BT_FIELD(total2, k);
    };
#pragma unroll
    for (int k = 0; k < G::PHASE; ++k) scatter(k, run0);
    const uint32_t first_total = row_start;
    if (staged) {
#pragma unroll
        for (int k = G::PHASE; k < R; ++k) scatter(k, run0);
    }

    if (dense_early) store_dense();

    // The wait for the tile's prefix, the index in the value array of its first value: by the first wave, or by all.
    uint32_t polls = 0;
    bool complete = false;
    uint64_t tile_g0;
    const auto itself = [&]() { return prefix_from_input<S, R, KEEP>(in, tile, threshold_f, threshold, lane_number()); };
    // Algorithm 2's j at the start of this tile, for bt_decompress_indexed; the index has the tiles of kRows rows
    const auto store_index = [&](const uint64_t j) __attribute__((always_inline)) {
        uint64_t *const index = job.index(sl.item);
        constexpr uint32_t kPerEntry = kRows / R;
        if (index != nullptr && tile % kPerEntry == 0) index[tile / kPerEntry] = j;
    };
    if constexpr (kQuarters) {
        const bool last = slot + 1 == n_slots;
        const uint32_t mine = wait_for_quarter(ws, slot, last, ep.cur, wave, polls);
        if (lane_number() == 0) s_found[wave] = mine;
        lds_barrier();
        tile_g0 = add_quarters(ws, s_found, last, complete, itself);
        complete = complete && wave == 0;
        if (wave == 0 && lane_number() == 0) store_index(tile_g0);
    } else {
        if (wave == 0) {
            const uint64_t v = DIRECT ? wait_for_counts(ws, slot, n_slots, ep.cur, polls, complete, itself) : wait_for_prefix(ws, slot, n_slots, ep.cur, polls, itself);
            if (lane_number() == 0) {
                s_tile_prefix = v;
                store_index(v);
            }
        }
        lds_barrier();
        tile_g0 = uniform64(s_tile_prefix);
    }
    BT_TL(slot, 2);
    BT_TL_VALUE(slot, 5, polls);
    if (!words_early) store_words();
    if (DENSE && !dense_early) store_dense();

    // (5)
    const uint64_t values_cap = job.cap(sl.item);
    // capacity clamp: never write at or beyond values_cap
    const auto room = [&](const uint64_t g0, const uint32_t cnt) {
        return g0 >= values_cap ? 0u : values_cap - g0 < cnt ? (uint32_t)(values_cap - g0) : cnt;
    };
    char *const values = static_cast<char *>(job.values(sl.item));
    if (staged) {
        run_store<S, kBlock, G::STAGE, false>(s_stage, values + tile_g0 * S, room(tile_g0, tile_total), wave * kWaveSize + lane_number());
    } else {
        unsigned char *const strip = s_stage + wave * kStrip;
        const uint64_t g0 = tile_g0 + before_wave, g1 = g0 + first_total;
        run_store<S, kWaveSize, G::PHASE * G::ROW * S, false>(strip, values + g0 * S, room(g0, first_total), lane_number());
        wave_lds_sync();                // the first phase's reads are done before the strip is reused
        row_start = 0;
        const int pad = (int)(reinterpret_cast<uintptr_t>(values + g1 * S) & (kVecBytes - 1));
#pragma unroll
        for (int k = G::PHASE; k < R; ++k) scatter(k, wave * kStrip + pad);
        wave_lds_sync();
        run_store<S, kWaveSize, G::PHASE * G::ROW * S, true>(strip, values + g1 * S, room(g1, row_start), lane_number());
    }
    // Without a scanner the last tile ends the call, when nothing of its own waits any more.  (Ended before its values were
    // written, with the header's count of calls read only then, it was a microsecond behind the others.  With both, us: fp32 12.5 k
    // elements 4.3 -> 3.9, 60 k 4.5 -> 4.1, 201 k 5.0 -> 4.7, bf16 60 k 4.8 -> 4.3, fp64 60 k 5.0 -> 4.4, fp32 activation call on 12.5 k 4.5 -> 4.2.)
    if (DIRECT && complete && lane_number() == 0) {
        store_nnz(job.nnz(0), tile_g0 + tile_total);
        // every slot's workgroup has published its count by now, hence has read the header: advance it
        header_finish(reinterpret_cast<uint32_t *>(ws), n_slots, ep.cur, ep.calls);
    }
    BT_TL(slot, 3);
}

// ---- Algorithm 2: bitmap -> dense ---------------------------------------------------------

// The reverse of run_store in two steps, so that the loads of several phases can be in
// flight together: strip_fetch issues the loads of values[g0, g0 + cnt) into
// registers, strip_commit later writes them into the wave's LDS strip, LDS element
// pad + i being global element g0 + i (pad lines LDS byte 0 up with a 16-byte boundary
// of the global buffer).  A phase of four rows holds at most PHASE * ROW elements, i.e. 257 aligned
// vectors: the inner ones (at most 255, all fully inside the range) go PHASE to a
// lane; of the first and the last vector, lane j < E takes element j of the first
// and lane E + j element j of the last, each only if it lies inside the range.
template <int S> struct Fetched {
    uint4 inner[Geo<S>::PHASE];
    typename std::conditional<S == 8, uint64_t, uint32_t>::type edge;
};

template <int S>
__device__ __forceinline__ void strip_fetch(const char *g0_ptr, const uint32_t pad, const uint32_t cnt, const int lane,
                                            Fetched<S> &f) {
    constexpr int E = Geo<S>::E;
    constexpr int PHASE = Geo<S>::PHASE;
    static_assert(PHASE * Geo<S>::ROW / E + 1 <= 2 + PHASE * kWaveSize, "a phase must fit PHASE inner vectors per lane");
    const char *gvec = g0_ptr - (size_t)pad * S;
    const uint32_t hi_valid = pad + cnt;
    const uint32_t n_vec = cnt ? (hi_valid + E - 1) / E : 0;
#pragma unroll
    for (int i = 0; i < Geo<S>::PHASE; ++i) {
        const uint32_t v = 1u + (uint32_t)lane + (uint32_t)kWaveSize * i;
        f.inner[i] = make_uint4(0, 0, 0, 0);
        if (v + 1 < n_vec) f.inner[i] = stream_load<kDecompressNtLoad>(reinterpret_cast<const uint4 *>(gvec + (size_t)v * kVecBytes));
    }
    f.edge = 0;
    if (lane < 2 * E && n_vec != 0) {
        const uint32_t e = lane < E ? (uint32_t)lane : (n_vec - 1) * E + (uint32_t)(lane - E);
        const bool wanted = e >= pad && e < hi_valid && (lane < E || n_vec > 1);
        if (wanted) {
            if (S == 8) f.edge = reinterpret_cast<const uint64_t *>(gvec)[e];
            else if (S == 4) f.edge = reinterpret_cast<const uint32_t *>(gvec)[e];
            else f.edge = reinterpret_cast<const uint16_t *>(gvec)[e];
        }
    }
}

template <int S>
__device__ __forceinline__ void strip_commit(unsigned char *strip, const uint32_t pad, const uint32_t cnt, const int lane,
                                             const Fetched<S> &f) {
    constexpr int E = Geo<S>::E;
    const uint32_t hi_valid = pad + cnt;
    const uint32_t n_vec = cnt ? (hi_valid + E - 1) / E : 0;
#pragma unroll
    for (int i = 0; i < Geo<S>::PHASE; ++i) {
        const uint32_t v = 1u + (uint32_t)lane + (uint32_t)kWaveSize * i;
        if (v + 1 < n_vec) *reinterpret_cast<uint4 *>(strip + (size_t)v * kVecBytes) = f.inner[i];
    }
    if (lane < 2 * E && n_vec != 0) {
        const uint32_t e = lane < E ? (uint32_t)lane : (n_vec - 1) * E + (uint32_t)(lane - E);
        const bool wanted = e >= pad && e < hi_valid && (lane < E || n_vec > 1);
        if (wanted) {
            if (S == 8) reinterpret_cast<uint64_t *>(strip)[e] = f.edge;
            else if (S == 4) reinterpret_cast<uint32_t *>(strip)[e] = (uint32_t)f.edge;
            else reinterpret_cast<uint16_t *>(strip)[e] = (uint16_t)f.edge;
        }
    }
}

// Restoration of one wave's quarter of a tile, where the scan tells the tile's place (without it: load_bits and what follows it):
//   quarter_load    asks for the bitmap words of the quarter, each once (lane l: words l * QPL ...);
//   restore_ranks   counts them, running sum over the lanes, and hands every lane the words and ranks of its rows
//                   (Algorithm 2's counter j inside the quarter) through LDS;
//   restore_fetch   given j at the start of the tile, asks for the wave's values;
//   restore_store   puts the values into the LDS strip, expands them by rank (a value where
//                   the bit is set, +0 where it is clear) and stores the dense quarter tile.
// (Read once per row by the lanes that share a word, and ranked by row sums, they cost a wave eight loads of 32 bytes,
// which keep the address units busy before anything else can start, and four times the DPP steps.  Measured, before /
// after, us: fp32 25.7 M 27.0 / 26.7, 206 M 214 / 212, fp16 206 M at 5 % 142.8 / 141.7.)
// (fetch_values, commit_values and expand_row of the restoration without the scan are three of these steps again, for a workgroup
// instead of a wave.  As one set of functions for both, or with the expansion alone shared, this kernel is scheduled otherwise and
// mostly slower.  Measured, us, as it is / one set / expansion shared: bf16 3 M elements at 50 % zeros 6.75 / 6.81 / 6.79, the 49 tensors
// of a ResNet-50 at one image in bf16, 70 % zeros, 10.89 / 10.97 / 10.98, fp64 25.7 M 59.0 / 59.6 / 59.1, fp32 100 M 105.6 / 105.5 / 105.8.)
template <int S> struct Quarter { uint32_t w[Geo<S>::QPL]; };

// Words at or beyond the bitmap's end read as 0, bits at or beyond n are cleared (Algorithm 2 visits n bits).
template <int S>
__device__ __forceinline__ Quarter<S> quarter_load(const uint32_t *bitmap, const uint64_t n, const uint32_t tile, const int lane, const int wave) {
    using G = Geo<S>;
    static_assert(G::QPL <= 2, "one load");
    typedef uint32_t word2 __attribute__((ext_vector_type(2), aligned(4)));      // (the bitmap is 4-byte aligned)
    const uint64_t first = (uint64_t)tile * G::TILE_WORDS + (uint64_t)wave * G::WAVE_WORDS;
    const bool full = (uint64_t)(tile + 1) * G::TILE <= n;
    Quarter<S> q;
#pragma unroll
    for (int j = 0; j < G::QPL; ++j) q.w[j] = 0;
    if (__builtin_expect(full, 1)) {
        if (G::QPL == 2) {
            const word2 v = *reinterpret_cast<const word2 *>(bitmap + first + 2 * lane);
            q.w[0] = v.x;
            q.w[G::QPL - 1] = v.y;
        } else if (G::WAVE_WORDS >= kWaveSize || lane < G::WAVE_WORDS) {
            q.w[0] = bitmap[first + lane];
        }
    } else {
        const uint64_t n_words = (n + 31) >> 5;      // (at least one)
#pragma unroll
        for (int j = 0; j < G::QPL; ++j) {
            const uint64_t wi = first + (uint32_t)(lane * G::QPL + j);
            q.w[j] = bitmap[wi < n_words ? wi : n_words - 1];
        }
#pragma unroll
        for (int j = 0; j < G::QPL; ++j) {
            const uint64_t wi = first + (uint32_t)(lane * G::QPL + j);
            if (lane * G::QPL + j >= G::WAVE_WORDS || wi >= n_words) q.w[j] = 0;
            if (wi + 1 == n_words && (n & 31) != 0) q.w[j] &= (1u << (uint32_t)(n & 31)) - 1u;
        }
    }
    return q;
}

template <int S> struct Restoring {            // a quarter tile between restore_ranks and restore_store
    static constexpr int PHASES = kRows / Geo<S>::PHASE;
    uint32_t mp[Geo<S>::MW], rank2[kRows / 2];          // ranks inside the quarter, two rows to a register
    uint32_t before[PHASES + 1];                       // set bits of the quarter before each phase, and all of them
    Fetched<S> fetched[PHASES];
    uint32_t pads[PHASES], cnts[PHASES];
};

// (1) this lane's bits of the bitmap (G lanes take E bits each of one word), and Algorithm 2's counter j as ranks.  Returns the
//     set bits of this wave's quarter of the tile.  `strip`: the wave's LDS, free until the values are put into it.
template <int S>
__device__ __forceinline__ uint32_t restore_ranks(const Quarter<S> &q, unsigned char *strip, const int lane, Restoring<S> &r) {
    using G = Geo<S>;
    constexpr int E = G::E;
    static_assert(8 * G::WAVE_WORDS <= G::LDS_WAVE && G::WAVE < 65536, "a word and its rank per entry; ranks in 16 bits");
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < G::QPL; ++j) mine += (uint32_t)__popc(q.w[j]);
    const uint32_t incl = wave_inclusive_sum(mine);
    uint32_t rank = incl - mine;
#pragma unroll
    for (int ph = 0; ph < Restoring<S>::PHASES; ++ph)       // the lane that holds the phase's first word
        r.before[ph] = (uint32_t)__builtin_amdgcn_readlane((int)rank, ph * G::PHASE * G::WPR / G::QPL);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    r.before[Restoring<S>::PHASES] = total;
    bt_u2 *const entries = reinterpret_cast<bt_u2 *>(strip);
    if (G::WAVE_WORDS >= kWaveSize || lane < G::WAVE_WORDS) {
#pragma unroll
        for (int j = 0; j < G::QPL; ++j) {
            entries[lane * G::QPL + j] = bt_u2{q.w[j], rank};
            rank += (uint32_t)__popc(q.w[j]);
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < G::MW; ++i) r.mp[i] = 0;
    const uint32_t shift = (uint32_t)E * (uint32_t)(lane % G::G);
    const uint32_t below = (1u << shift) - 1u;
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const bt_u2 e = entries[k * G::WPR + lane / G::G];
        r.mp[k / G::RPM] |= ((e.x >> shift) & ((1u << E) - 1u)) << (E * (k % G::RPM));
        const uint32_t at = e.y + (uint32_t)__popc(e.x & below);
        r.rank2[k / 2] = (k & 1) == 0 ? at : r.rank2[k / 2] | (at << 16);
    }
    wave_lds_sync();                    // the entries are read before the strip is used for values
    return total;
}

// (2) ask for the values of every phase (PHASE rows each), so that all of them are in flight together
template <int S>
__device__ __forceinline__ void restore_fetch(const void *__restrict__ values, const uint64_t values_cap, const uint64_t tile_j,
                                              const uint32_t before_wave, const int lane, Restoring<S> &r) {
    using G = Geo<S>;
    uint64_t g0 = tile_j + before_wave;                                   // Algorithm 2's j for this wave
#pragma unroll
    for (int ph = 0; ph < Restoring<S>::PHASES; ++ph) {
        r.cnts[ph] = r.before[ph + 1] - r.before[ph];
        const char *gsrc = static_cast<const char *>(values) + g0 * S;
        r.pads[ph] = (uint32_t)(reinterpret_cast<uintptr_t>(gsrc) & (kVecBytes - 1)) / S;
        const uint32_t phase_total = r.cnts[ph];
        // nothing at or beyond the capacity is read (an index that does not belong to the bitmap, a wait that ran out)
        if (g0 >= values_cap) r.cnts[ph] = 0;
        else if (values_cap - g0 < r.cnts[ph]) r.cnts[ph] = (uint32_t)(values_cap - g0);
        strip_fetch<S>(gsrc, r.pads[ph], r.cnts[ph], lane, r.fetched[ph]);
        g0 += phase_total;
    }
}

template <int S>
__device__ __forceinline__ void restore_store(const Restoring<S> &r, const uint64_t n, void *__restrict__ out, const uint32_t tile,
                                              unsigned char *strip, const int lane, const int wave) {
    using G = Geo<S>;
    constexpr int E = G::E;
    const uint64_t wave_e0 = (uint64_t)tile * G::TILE + (uint64_t)wave * G::WAVE;
    const bool full = (uint64_t)(tile + 1) * G::TILE <= n;
#pragma unroll
    for (int ph = 0; ph < Restoring<S>::PHASES; ++ph) {
        if (ph != 0) wave_lds_sync();   // the previous phase's reads are done before the strip is reused
        strip_commit<S>(strip, r.pads[ph], r.cnts[ph], lane, r.fetched[ph]);
        wave_lds_sync();
        const uint32_t base = r.pads[ph] - r.before[ph];
#pragma unroll
        for (int k = ph * G::PHASE; k < (ph + 1) * G::PHASE; ++k) {
            uint32_t at = base + BT_FIELD(r.rank2, k);
            const uint32_t mk = BT_MASK(S, r.mp, k);
            uint32_t d[4] = {0, 0, 0, 0};
            // every lane reads at its running rank whether the bit is set or not (the index stays inside the strip)
            // and a select drops what a cleared bit read
            if (S == 8) {
                const uint64_t *l = reinterpret_cast<const uint64_t *>(strip);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const uint32_t keep = (mk >> j) & 1u;
                    const uint64_t v = l[at];
                    d[2 * j] = keep ? (uint32_t)v : 0u;
                    d[2 * j + 1] = keep ? (uint32_t)(v >> 32) : 0u;
                    at += keep;
                }
            } else if (S == 4) {
                const uint32_t *l = reinterpret_cast<const uint32_t *>(strip);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t keep = (mk >> j) & 1u;
                    const uint32_t v = l[at];
                    d[j] = keep ? v : 0u;
                    at += keep;
                }
            } else {
                const uint16_t *l = reinterpret_cast<const uint16_t *>(strip);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const uint32_t keep = (mk >> j) & 1u;
                    const uint32_t v = l[at];
                    d[j >> 1] |= (keep ? v : 0u) << (16 * (j & 1));
                    at += keep;
                }
            }
            const uint64_t e0 = wave_e0 + (uint64_t)k * G::ROW + (uint64_t)lane * E;
            const uint4 o = make_uint4(d[0], d[1], d[2], d[3]);
            if (full) stream_store<kDecompressNtStore>(reinterpret_cast<uint4 *>(static_cast<char *>(out) + e0 * S), o);
            else store_vec_guarded<S>(out, e0, n, o);
        }
    }
}

// What a restoring wave does when the scanner's answer for its tile does not come: it counts the set
// bits of the tensor's bitmap before the tile itself.  Slow (the whole bitmap up to the tile), but it
// needs nothing from any other workgroup.  Every bit before a tile is a bit of the tensor, so no mask.
template <int S>
__device__ __noinline__ uint64_t prefix_from_bitmap(const uint32_t *__restrict__ bitmap, const uint32_t tile, const int lane) {
    const uint64_t words = (uint64_t)tile * Geo<S>::TILE_WORDS;
    uint64_t mine = 0;
    for (uint64_t w = (uint32_t)lane; w < words; w += kWaveSize) mine += (uint32_t)__popc(bitmap[w]);
#pragma unroll
    for (int d = 1; d < kWaveSize; d <<= 1) mine += __shfl_xor((unsigned long long)mine, d, kWaveSize);
    return uniform64(mine);
}

// bt_decompress and bt_decompress_batch: workgroup 0 is the scanner (one wave of it), workgroup 1 + t
// restores slot t.  A tile's count depends
// on the bitmap alone: every wave turns its bitmap words into masks and ranks, whose totals are the
// wave's share of the count; the workgroup adds the shares up and publishes the count; then the first
// wave waits for the tile's prefix, every wave fetches its values, expands and stores them, and the
// workgroup ends.
//
// Why a workgroup per tile and no loop over tiles.  A wave that has issued its stores
// is gone (nothing waits for them to land) and the next workgroup takes its place, whereas a wave that
// went on to a next tile would, on this hardware, wait for its own stores whenever it waits for that
// tile's loads (one counter tracks both, in order).  Two thirds of a restoration's traffic are stores;
// kernels that loop measured 10 to 25 % slower, with or without the next tile's loads in flight.
//
// Forward progress does not rest on the order in which workgroups are started.  A workgroup publishes
// its count before it waits for anything, and one whose prefix has not come after kPatience polls
// stops waiting and counts the bitmap itself (prefix_from_bitmap): so every workgroup that has been
// started ends, whatever the others do, and every workgroup is started in the end.
//
// MODE kScannedSoon: the header is asked for behind the bitmap words instead of waited for before them.  That takes a round trip off the
// start of a launch; where workgroups come and go, one that starts sooner also adds to what the stores compete with.  The line, at 1024
// tiles for all elements, is where the 16-bit ones stop to gain; wider ones gain a little beyond it too.  Measured, us, kScanned / this: fp32
// 4.5 M elements (549 tiles) 8.9 / 8.7, 8 M 11.9 / 11.7, fp64 3.2 M 10.9 / 10.4, bf16 9 M 9.5 / 9.2, 15 M (916) 11.9 / 11.9; beyond the line bf16 21 M
// (1282) 14.2 / 14.6, 33 M 19.6 / 19.9, 25.7 M at 95 % zeros 14.0 / 13.8, fp32 9 M (1099) 12.9 / 12.7, 12.8 M 16.2 / 16.0, 20 M 22.4 / 22.0, 25.7 M 26.6 / 26.7,
// fp64 4.5 M (1099) 13.0 / 12.5, 6.4 M 16.4 / 15.9, 12.8 M 26.7 / 26.4.
// MODE kQuartered: launches on one tensor of up to kQuarterSlots tiles, without a scanner, whose tiles' waves read a quarter of the counts each
// as in compression (wait_for_quarter); the last tile ends the call.  Two workgroups a compute unit at most, so there are registers.
// Measured, us, with the scanner / this: fp32 2.2 M elements 7.1 / 6.7, 3.2 M 7.5 / 7.0, 4.2 M 7.9 / 7.3, at 5 % zeros 9.3 / 8.5; bf16 4.5 M
// 7.8 / 7.3, 6.4 M 8.0 / 7.4, 8.4 M 8.4 / 7.8, at 5 % 9.7 / 9.2; bf16 3.2 M (196 tiles) 6.6 / 6.6; fp64 2.1 M 7.4 / 8.4 (not done).
enum { kScanned, kScannedSoon, kQuartered };
template <int S, int MODE, class Job>
__global__ __launch_bounds__(kBlock, MODE == kQuartered ? 7 : kDecompressOcc) void decompress_kernel(const Job job, char *ws) {
    using G = Geo<S>;
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[kWaves * G::LDS_WAVE];
    __shared__ uint64_t s_tile_j;
    __shared__ uint32_t s_wave_total[kWaves], s_found[kWaves];
    const uint32_t n_slots = gridDim.x - (MODE == kQuartered ? 0u : 1u);
    if (MODE != kQuartered && blockIdx.x == 0) {
        if (threadIdx.x < kWaveSize && !epoch_of(read_header(ws)).failed) scan_counts<2>(ws, job);
        return;
    }
    BT_TL_INIT;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t slot = blockIdx.x - (MODE == kQuartered ? 0u : 1u);
    // The header while the bitmap words are on their way, as in compression, or (MODE = kScanned) before them.
    HeaderWords header;
    if (MODE == kScanned) {
        header = read_header(ws);
        if (__builtin_expect(epoch_of(header).failed, 0)) {
            if (lane == 0) s_wave_total[wave] = kWaveFailed;
            lds_barrier();
            return;
        }
    }
    const Slot sl = job.at(slot);
    // everything else waits for these
    const uint32_t *const bitmap = job.bitmap(sl.item);
    const uint64_t n = job.n(sl.item);
    const Quarter<S> quarter = quarter_load<S>(bitmap, n, sl.tile, lane, wave);
    if (MODE != kScanned) {
        asm volatile("" ::: "memory");
        header = read_header(ws);
    }
    BT_TL(slot, 0);
    // masks and ranks; what they add up to is this wave's share of the tile's count
    Restoring<S> r;
    unsigned char *const strip = s_stage + wave * G::LDS_WAVE;
    const uint32_t wave_total = restore_ranks<S>(quarter, strip, lane, r);
    const Epoch ep = epoch_of(header);
    if (lane == 0) s_wave_total[wave] = ep.failed ? kWaveFailed : wave_total;
    lds_barrier();                      // also: every wave has read the header before the first wave publishes anything
    if (any_wave_failed(s_wave_total)) return;
    uint32_t before_wave = 0, tile_total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_wave_total[w];
        if (w < wave) before_wave += c;
        tile_total += c;
    }
    before_wave = uniform32(before_wave);       // the same in every lane: tell the compiler, so that addresses built on it stay scalar
    uint32_t polls = 0;
    if (tid == 0) ws_store32(ws_count(ws, slot, ep.cur), (tile_total + 1) | (Job::kMany && sl.tile == 0 ? kFirstTile : 0u));
    BT_TL(slot, 1);
    zero_previous(ws, ep, slot, n_slots);
    // Algorithm 2's counter j at the start of the tile: with a scanner the first wave asks (one poller a tile keeps the
    // traffic on the workspace's few lines low) and passes the answer on through LDS
    uint64_t tile_j;
    bool complete = false;
    if constexpr (MODE == kQuartered) {
        const bool last = slot + 1 == n_slots;
        const uint32_t mine = wait_for_quarter(ws, slot, last, ep.cur, wave, polls);
        if (lane == 0) s_found[wave] = mine;
        lds_barrier();
        // (not prefix_from_bitmap: a call that all waves may make costs the registers that live across it)
        tile_j = add_quarters(ws, s_found, last, complete, [&]() {
            uint32_t share = 0;
#pragma unroll 1
            for (uint32_t w = (uint32_t)lane_number(); w < sl.tile * (uint32_t)G::TILE_WORDS; w += kWaveSize) share += (uint32_t)__popc(bitmap[w]);
            return wave_total_of(share);
        });
    } else {
        if (wave == 0) {
            const uint64_t v = wait_for_prefix(ws, slot, n_slots, ep.cur, polls, [&]() { return prefix_from_bitmap<S>(bitmap, sl.tile, lane); });
            if (lane == 0) s_tile_j = v;
        }
        lds_barrier();
        tile_j = uniform64(s_tile_j);
    }
    BT_TL(slot, 2);
    restore_fetch<S>(job.values(sl.item), job.cap(sl.item), tile_j, before_wave, lane, r);
    restore_store<S>(r, n, job.out(sl.item), sl.tile, strip, lane, wave);
    if (MODE == kQuartered && complete && wave == 0 && lane == 0) header_finish(reinterpret_cast<uint32_t *>(ws), n_slots, ep.cur, ep.calls);
    BT_TL(slot, 3);
    BT_TL_VALUE(slot, 5, polls);
}

// ---- restoration without the scan ------------------------------------------------------------
//
// Restoration of a tile by a workgroup whose tile's place is known without a wait:
//   load_bits     a wave asks for the bitmap words of the whole tile, each once (lane l: words l * WPL ...);
//   rank_words    counts them, running sum over the lanes: every wave knows the rank of every word, so the waves need
//                 not meet for it;
//   rows_of       hands the lanes the words and ranks of the wave's rows (Algorithm 2's counter j inside the tile) through LDS;
//   fetch_values  given j at the start of the tile, asks for the values of one phase (PHASE rows of every wave), a contiguous run;
//   commit_values puts them into LDS, where all waves find them;
//   expand_row    a value where the bit is set, +0 where it is clear, by rank; 16-byte dense stores.
// The waves take the tile's rows in turn (of W waves, wave w rows w, w + W, ...): a phase is one contiguous piece of the tensor and of the
// values, and it is written from front to back.  When every wave had a quarter of the tile with a strip of LDS of its own, a phase
// was eight pieces, each with element-wise edges and partial cache lines of its own, written at four places at once.
// (With the scan it is the other way round: quarters publish their counts from a fourth of the loads, and the waves of a tile that
// has its prefix do not wait for each other.  Measured, us, quarters / this: fp32 3 M elements 7.5 / 7.7, 25.7 M 26.6 / 26.9, bf16 3 M
// 7.9 / 8.3, fp64 25.7 M 58.2 / 63.5.)

// Bits of words at or beyond the bitmap's end, and bits at or beyond n, are 0 (Algorithm 2 visits n bits).
template <int S, int R, int W = kWaves> struct TileBits { uint32_t w[Geo<S, R, W>::WPL]; };

template <int S, int R, int W = kWaves>
__device__ __forceinline__ TileBits<S, R, W> load_bits(const uint32_t *bitmap, const uint64_t n, const uint32_t tile, const int lane) {
    using G = Geo<S, R, W>;
    constexpr int WPL = G::WPL;
    typedef uint32_t words __attribute__((ext_vector_type(WPL), aligned(4)));      // (the bitmap is 4-byte aligned)
    const uint64_t first = (uint64_t)tile * G::TILE_WORDS;
    TileBits<S, R, W> b;
#pragma unroll
    for (int j = 0; j < WPL; ++j) b.w[j] = 0;
    if (__builtin_expect((uint64_t)(tile + 1) * G::TILE <= n, 1)) {
        if (G::TILE_WORDS >= kWaveSize || lane < G::TILE_WORDS) {
            const words v = *reinterpret_cast<const words *>(bitmap + first + lane * WPL);
#pragma unroll
            for (int j = 0; j < WPL; ++j) b.w[j] = v[j];
        }
    } else {
        // a tensor's last tile (n > tile * TILE): all loads at once, from clamped addresses
        const uint64_t left = ((n + 31) >> 5) - first;
        const uint32_t there = left < (uint64_t)G::TILE_WORDS ? (uint32_t)left : (uint32_t)G::TILE_WORDS;
        const uint32_t tail = left <= (uint64_t)G::TILE_WORDS && (n & 31) != 0 ? (1u << (uint32_t)(n & 31)) - 1u : ~0u;
#pragma unroll
        for (int j = 0; j < WPL; ++j) b.w[j] = bitmap[first + min((uint32_t)(lane * WPL + j), there - 1u)];
#pragma unroll
        for (int j = 0; j < WPL; ++j) {
            const uint32_t i = (uint32_t)(lane * WPL + j);
            b.w[j] &= i + 1u < there ? ~0u : i + 1u == there ? tail : 0u;
        }
    }
    return b;
}

// Set bits of the tile before the lane's first word, and before each phase and after the last one.
template <int S, int R, int W = kWaves> struct TileRanks {
    static constexpr int PHASES = R / Geo<S, R, W>::PHASE;
    uint32_t mine;
    uint32_t before[PHASES + 1];
};

template <int S, int R, int W = kWaves> __device__ __forceinline__ TileRanks<S, R, W> rank_words(const TileBits<S, R, W> &b) {
    using G = Geo<S, R, W>;
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < G::WPL; ++j) sum += (uint32_t)__popc(b.w[j]);
    const uint32_t incl = wave_inclusive_sum(sum);
    TileRanks<S, R, W> r;
    r.mine = incl - sum;
#pragma unroll
    for (int ph = 0; ph < TileRanks<S, R, W>::PHASES; ++ph)       // (the lane that holds the phase's first word)
        r.before[ph] = (uint32_t)__builtin_amdgcn_readlane((int)r.mine, ph * W * G::PHASE * G::WPR / G::WPL);
    r.before[TileRanks<S, R, W>::PHASES] = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    return r;
}

// The lane's bits of K rows of its wave (G lanes take E bits each of one word), and Algorithm 2's j as ranks in the tile.
template <int S, int K> struct Rows {
    uint32_t mp[Geo<S, K>::MW], rank2[K / 2];          // two rows' ranks to a register
};

// The wave's rows among the tile's rows [first, first + W * K).  `entries`: room for their words, a pair each; a wave writes and reads
// those of its own rows only.
template <int S, int R, int K, int W = kWaves>
__device__ __forceinline__ Rows<S, K> rows_of(const TileBits<S, R, W> &b, const TileRanks<S, R, W> &r, const int first, bt_u2 *entries, const int lane, const int wave) {
    using G = Geo<S, R, W>;
    constexpr int E = G::E;
    static_assert(G::TILE < 65536, "ranks in 16 bits");
    uint32_t rank = r.mine;
#pragma unroll
    for (int j = 0; j < G::WPL; ++j) {
        const int i = lane * G::WPL + j;
        const int row = i / G::WPR;
        const bool asked = K == R || (unsigned)(row - first) < (unsigned)(W * K);
        if (asked && row % W == wave && (G::TILE_WORDS >= kWaveSize || lane < G::TILE_WORDS)) entries[i - first * G::WPR] = bt_u2{b.w[j], rank};
        rank += (uint32_t)__popc(b.w[j]);
    }
    wave_lds_sync();
    Rows<S, K> rows;
#pragma unroll
    for (int i = 0; i < Geo<S, K>::MW; ++i) rows.mp[i] = 0;
    const uint32_t shift = (uint32_t)E * (uint32_t)(lane % G::G);
    const uint32_t below = (1u << shift) - 1u;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const bt_u2 e = entries[(k * W + wave) * G::WPR + lane / G::G];
        rows.mp[k / G::RPM] |= ((e.x >> shift) & ((1u << E) - 1u)) << (E * (k % G::RPM));
        const uint32_t at = e.y + (uint32_t)__popc(e.x & below);
        rows.rank2[k / 2] = (k & 1) == 0 ? at : rows.rank2[k / 2] | (at << 16);
    }
    return rows;
}

// The values of one phase on their way to LDS, whose element pad + i is the phase's i-th (pad lines LDS byte 0 up with a 16-byte
// boundary of the value array).  They are at most PHASE * W * kWaveSize + 1 aligned vectors: the inner ones, all fully inside the
// range, go PHASE to a thread; of the first and the last vector, thread j < E takes element j of the first and thread
// E + j element j of the last, each only if it lies inside the range.
template <int S, int R, int W = kWaves> struct TileValues {
    uint4 inner[Geo<S, R, W>::PHASE];
    typename std::conditional<S == 8, uint64_t, uint32_t>::type edge;
    uint32_t pad, end;      // elements of LDS [pad, end) are values
};

// Is there an edge element for thread `tid`, and which?
template <int S, int R, int W = kWaves> __device__ __forceinline__ bool edge_of(const TileValues<S, R, W> &f, const int tid, uint32_t &at) {
    constexpr int E = Geo<S, R, W>::E;
    const uint32_t vecs = (f.end + E - 1) / E;
    at = tid < E ? (uint32_t)tid : (vecs - 1) * E + (uint32_t)(tid - E);
    return tid < 2 * E && f.end != f.pad && at >= f.pad && at < f.end && (tid < E || vecs > 1);
}

// j: position of the phase's first value; nothing at or beyond the capacity is read (an index that does not belong to the
// bitmap, a wait that ran out).
template <int S, int R, int W = kWaves>
__device__ __forceinline__ TileValues<S, R, W> fetch_values(const void *__restrict__ values, const uint64_t values_cap, const uint64_t j, uint32_t count, const int tid) {
    using G = Geo<S, R, W>;
    constexpr int E = G::E;
    if (j >= values_cap) count = 0;
    else if (values_cap - j < count) count = (uint32_t)(values_cap - j);
    const char *const src = static_cast<const char *>(values) + j * S;
    TileValues<S, R, W> f;
    f.pad = (uint32_t)(reinterpret_cast<uintptr_t>(src) & (kVecBytes - 1)) / S;
    f.end = f.pad + count;
    const char *const vec = src - (size_t)f.pad * S;
#pragma unroll
    for (int i = 0; i < G::PHASE; ++i) {
        const uint32_t v = 1u + (uint32_t)tid + (uint32_t)(W * kWaveSize) * i;
        f.inner[i] = make_uint4(0, 0, 0, 0);
        if ((v + 1) * E < f.end) f.inner[i] = stream_load<kDecompressNtLoad>(reinterpret_cast<const uint4 *>(vec + (size_t)v * kVecBytes));
    }
    f.edge = 0;
    uint32_t at;
    if (edge_of<S, R, W>(f, tid, at)) {
        if (S == 8) f.edge = reinterpret_cast<const uint64_t *>(vec)[at];
        else if (S == 4) f.edge = reinterpret_cast<const uint32_t *>(vec)[at];
        else f.edge = reinterpret_cast<const uint16_t *>(vec)[at];
    }
    return f;
}

template <int S, int R, int W = kWaves>
__device__ __forceinline__ void commit_values(unsigned char *stage, const TileValues<S, R, W> &f, const int tid) {
    using G = Geo<S, R, W>;
    constexpr int E = G::E;
#pragma unroll
    for (int i = 0; i < G::PHASE; ++i) {
        const uint32_t v = 1u + (uint32_t)tid + (uint32_t)(W * kWaveSize) * i;
        if ((v + 1) * E < f.end) *reinterpret_cast<uint4 *>(stage + (size_t)v * kVecBytes) = f.inner[i];
    }
    uint32_t at;
    if (edge_of<S, R, W>(f, tid, at)) {
        if (S == 8) reinterpret_cast<uint64_t *>(stage)[at] = f.edge;
        else if (S == 4) reinterpret_cast<uint32_t *>(stage)[at] = (uint32_t)f.edge;
        else reinterpret_cast<uint16_t *>(stage)[at] = (uint16_t)f.edge;
    }
}

// 16 bytes of the dense tensor.  The lane reads at its running rank whether a bit is set or not (the place stays inside
// the staging area) and a select drops what a cleared bit read.
template <int S> __device__ __forceinline__ uint4 expand_row(const unsigned char *stage, uint32_t at, const uint32_t mk) {
    uint32_t d[4] = {0, 0, 0, 0};
    if (S == 8) {
        const uint64_t *l = reinterpret_cast<const uint64_t *>(stage);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const uint32_t keep = (mk >> j) & 1u;
            const uint64_t v = l[at];
            d[2 * j] = keep ? (uint32_t)v : 0u;
            d[2 * j + 1] = keep ? (uint32_t)(v >> 32) : 0u;
            at += keep;
        }
    } else if (S == 4) {
        const uint32_t *l = reinterpret_cast<const uint32_t *>(stage);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t keep = (mk >> j) & 1u;
            const uint32_t v = l[at];
            d[j] = keep ? v : 0u;
            at += keep;
        }
    } else {
        const uint16_t *l = reinterpret_cast<const uint16_t *>(stage);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t keep = (mk >> j) & 1u;
            const uint32_t v = l[at];
            d[j >> 1] |= (keep ? v : 0u) << (16 * (j & 1));
            at += keep;
        }
    }
    return make_uint4(d[0], d[1], d[2], d[3]);
}

// The wave's rows [k0, k0 + PHASE) of `rows`, which are rows first + k * W + wave of the tile; `before`: set bits of the tile before the phase.
template <int S, int R, int K, int W = kWaves>
__device__ __forceinline__ void expand_phase(const Rows<S, K> &rows, const int k0, const int first, const TileValues<S, R, W> &f, const uint32_t before,
                                             const unsigned char *stage, void *__restrict__ out, const uint64_t n, const uint32_t tile, const int lane,
                                             const int wave) {
    using G = Geo<S, R, W>;
    const uint64_t tile_e0 = (uint64_t)tile * G::TILE;
    const bool full = tile_e0 + G::TILE <= n;
#pragma unroll
    for (int k = k0; k < k0 + G::PHASE; ++k) {
        const uint4 o = expand_row<S>(stage, f.pad - before + BT_FIELD(rows.rank2, k), BT_MASK(S, rows.mp, k));
        const uint64_t e0 = tile_e0 + (uint64_t)((uint32_t)(first + k * W + wave) * G::ROW + (uint32_t)lane * G::E);
        if (full) stream_store<kDecompressNtStore>(reinterpret_cast<uint4 *>(static_cast<char *>(out) + e0 * S), o);
        else store_vec_guarded<S>(out, e0, n, o);
    }
}

// One thread's share of the set bits in the first `words` words of the bitmap (a whole number of 16-byte vectors), the
// workgroup's threads taking a vector each in turn.  kAhead loads are in flight together.
template <int THREADS>
__device__ __forceinline__ uint32_t count_share(const uint32_t *__restrict__ bitmap, const uint32_t words, const int tid) {
    typedef uint32_t word4 __attribute__((ext_vector_type(4), aligned(4)));      // (the bitmap is 4-byte aligned)
    constexpr uint32_t kAhead = 8;
    uint32_t count = 0;
    for (uint32_t first = 0; first < words; first += 4u * THREADS * kAhead) {
        word4 v[kAhead];
#pragma unroll
        for (uint32_t i = 0; i < kAhead; ++i) {
            const uint32_t w = first + 4u * (THREADS * i + (uint32_t)tid);
            v[i] = word4{0, 0, 0, 0};
            if (w < words) v[i] = *reinterpret_cast<const word4 *>(bitmap + w);
        }
#pragma unroll
        for (uint32_t i = 0; i < kAhead; ++i)
            count += (uint32_t)(__popc(v[i].x) + __popc(v[i].y) + __popc(v[i].z) + __popc(v[i].w));
    }
    return count;
}


// Small tensors (see bt_decompress): no scanner and nothing published.  Every workgroup of W waves counts the bitmap before
// its tile itself, all its threads together while its own words are on their way: what sits in the caches, against
// four hops through memory.  Bound by that count, a compute unit's reads through its first-level cache: eight waves halve what is
// read for a tensor, and ask for twice as much at once.  The call leaves the workspace's entries alone.  (With each wave restoring a quarter of the tile,
// us: fp32 30 k elements 3.1, 201 k 3.1, 700 k 4.5, bf16 201 k 3.2; now 2.9, 2.9, 4.3, 3.1.)
template <int S, int R, int W = kWaves>
__global__ __launch_bounds__(W * kWaveSize, kDecompressOcc) void decompress_small_kernel(const DecompressOne job, char *ws) {
    using G = Geo<S, R, W>;
    static_assert(TileRanks<S, R, W>::PHASES == 1, "one phase");
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[G::LDS_TILE];
    __shared__ bt_u2 s_entries[G::TILE_WORDS];
    __shared__ uint32_t s_wave_before[W], s_wave_total[W];
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tile = blockIdx.x;
    uint32_t *const hdr = reinterpret_cast<uint32_t *>(ws);
    const uint32_t calls = hdr[kHdrCalls], error = hdr[kHdrError];
    const uint32_t *const bitmap = job.bitmap(0);
    const uint64_t n = job.n(0);
    const TileBits<S, R, W> bits = load_bits<S, R, W>(bitmap, n, tile, lane);
    const uint32_t before_share = count_share<W * kWaveSize>(bitmap, tile * G::TILE_WORDS, tid);
    const TileRanks<S, R, W> ranks = rank_words<S, R, W>(bits);
    const Rows<S, R> rows = rows_of<S, R, R, W>(bits, ranks, 0, s_entries, lane, wave);
    const uint32_t incl = wave_inclusive_sum(before_share);
    if (lane == kWaveSize - 1) s_wave_before[wave] = incl;
    if (lane == 0) s_wave_total[wave] = uniform32(error) != 0 ? kWaveFailed : 0u;
    lds_barrier();                      // also: every wave has read the header before the first workgroup's first wave counts the call
    if (any_wave_failed(s_wave_total)) return;
    uint64_t tile_j = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) tile_j += s_wave_before[w];
    tile_j = uniform64(tile_j);
    if (tile == 0 && tid == 0) hdr[kHdrCalls] = calls + 1u;
    const TileValues<S, R, W> f = fetch_values<S, R, W>(job.values(0), job.cap(0), tile_j, ranks.before[1], tid);
    commit_values<S, R, W>(s_stage, f, tid);
    lds_barrier();
    expand_phase<S, R, R, W>(rows, 0, 0, f, 0, s_stage, job.out(0), n, tile, lane, wave);
}

// bt_decompress_indexed and its batched form: two workgroups per slot, one for each phase of its tile, and nothing else.
// Algorithm 2's j at the start of the tile comes from the tile index; what the tile's first half holds a wave of the second
// counts from the same words.
//
// What bounds it: the memory system on large tensors, the chain index and words, values, stores on small ones, so the less a workgroup
// has to do one after the other the better: half a tile, rows of all waves written front to back.  Measured, a workgroup per tile
// whose waves restore a quarter each / this, us: one tensor, fp32 3 M elements at 50 % zeros 4.3 / 3.8, 100 M 101.6 / 98.9, at 95 %
// 74.8 / 70.0; bf16 1 M 5.9 / 3.8, 25.7 M 16.2 / 13.2, 100 M 57.2 / 51.9, fp16 206 M at 95 % 71.8 / 65.6; fp64 100 M 200.9 / 195.9; the
// 49 tensors of a ResNet-50, fp32 at 1 / 4 / 64 images, 50 %, 12.9 / 10.9, 43.2 / 38.1, 641.7 / 613.9, at 64 images and 95 % 526 / 474, bf16 at
// 1 image 13.1 / 7.3.  Tiles of two rows instead of four: fp32 100 M at 95 % 60.1, but 106 at 50 %; six workgroups a compute unit
// instead of eight: 612.6 instead of 624.5 on the fp32 set at 50 %, 527 instead of 484 at 85 %.
template <int S, class Job>
__global__ __launch_bounds__(kBlock, kDecompressOcc) void decompress_indexed_kernel(const Job job, const uint32_t first_slot) {
    constexpr int R = kRows;
    using G = Geo<S, R>;
    static_assert(TileRanks<S, R>::PHASES == 2, "a workgroup per phase");
    __shared__ __attribute__((aligned(16))) unsigned char s_stage[G::LDS_TILE];
    __shared__ bt_u2 s_entries[G::TILE_WORDS / 2];
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Slot sl = job.at(first_slot + blockIdx.x / 2);
    const uint32_t half = blockIdx.x % 2;
    const uint64_t n = job.n(sl.item);
    if ((uint64_t)sl.tile * G::TILE + half * (G::TILE / 2) >= n) return;
    const uint64_t tile_j = job.tile_index(sl.item)[sl.tile];
    const TileBits<S, R> bits = load_bits<S, R>(job.bitmap(sl.item), n, sl.tile, lane);
    const TileRanks<S, R> ranks = rank_words<S, R>(bits);
    const uint32_t before = half != 0 ? ranks.before[1] : 0u;
    const uint32_t count = half != 0 ? ranks.before[2] - ranks.before[1] : ranks.before[1];
    const TileValues<S, R> f = fetch_values<S, R>(job.values(sl.item), job.cap(sl.item), tile_j + before, count, tid);
    const int first_row = (int)half * (kWaves * G::PHASE);
    const Rows<S, G::PHASE> rows = rows_of<S, R, G::PHASE>(bits, ranks, first_row, s_entries, lane, wave);
    commit_values<S, R>(s_stage, f, tid);
    lds_barrier();
    expand_phase<S, R, G::PHASE>(rows, 0, first_row, f, before, s_stage, job.out(sl.item), n, sl.tile, lane, wave);
}

// ---- ReLU backward from the bitmap -----------------------------------------------------------

// grad_in[i] = bit(i) ? grad_out[i] : +0.  Pure streaming: no scan, no LDS.  Each
// lane selects per element with the E bits that cover its 16-byte vector.  Bound by memory; NT: gradients are read past the
// caches (see bt_relu_backward_from_bitmap).
template <int S, bool NT>
__global__ __launch_bounds__(kBlock) void relu_backward_kernel(const uint32_t *__restrict__ bitmap,
                                                               const void *grad_out, const uint64_t n,
                                                               void *grad_in) {
    using G = Geo<S>;
    constexpr int E = G::E;
    constexpr int kR = kReluRows;                       // 16-byte vectors per lane
    constexpr int kTile = kBlock * kR * E;              // elements per block
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t n_words = (n + 31) >> 5;
    const uint64_t wave_e0 = (uint64_t)blockIdx.x * kTile + (uint64_t)wave * (kR * G::ROW);
    const bool full = ((uint64_t)blockIdx.x + 1) * kTile <= n;

    uint4 g[kR];
    uint32_t m[kR];
#pragma unroll
    for (int k = 0; k < kR; ++k) {
        const uint64_t e0 = wave_e0 + (uint64_t)k * G::ROW + (uint64_t)lane * E;
        if (full) {
            g[k] = stream_load<NT>(reinterpret_cast<const uint4 *>(static_cast<const char *>(grad_out) + e0 * S));
            m[k] = (bitmap[e0 >> 5] >> (uint32_t)(e0 & 31)) & ((1u << E) - 1u);
        } else {
            g[k] = load_vec_guarded<S>(grad_out, e0, n);
            m[k] = bitmap_bits<S>(bitmap, e0, n, n_words);
        }
    }
#pragma unroll
    for (int k = 0; k < kR; ++k) {
        const uint64_t e0 = wave_e0 + (uint64_t)k * G::ROW + (uint64_t)lane * E;
        uint32_t d[4] = {g[k].x, g[k].y, g[k].z, g[k].w};
        if (S == 8) {
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = (m[k] & (1u << (j >> 1))) ? d[j] : 0u;
        } else if (S == 4) {
#pragma unroll
            for (int j = 0; j < 4; ++j) d[j] = (m[k] & (1u << j)) ? d[j] : 0u;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t keep = ((m[k] & (1u << (2 * j))) ? 0x0000ffffu : 0u) |
                                      ((m[k] & (1u << (2 * j + 1))) ? 0xffff0000u : 0u);
                d[j] &= keep;
            }
        }
        const uint4 o = make_uint4(d[0], d[1], d[2], d[3]);
        if (full) stream_store<kReluNtStore>(reinterpret_cast<uint4 *>(static_cast<char *>(grad_in) + e0 * S), o);
        else store_vec_guarded<S>(grad_in, e0, n, o);
    }
}

// ---- ReLU and its bitmap ---------------------------------------------------------------------

// Which elements of the 16-byte vector ReLU keeps: the positive ones and NaNs, told from the bit pattern (as a signed number
// above 0, or as an unsigned one above that of minus infinity).
template <int S, int KEEP> __device__ __forceinline__ uint32_t relu_mask(const uint4 v) {
    const uint32_t d[4] = {v.x, v.y, v.z, v.w};
    uint32_t m = 0;
    if (S == 8) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint64_t b = ((uint64_t)d[2 * i + 1] << 32) | d[2 * i];
            m |= ((int64_t)b > 0 || b > 0xfff0000000000000ull ? 1u : 0u) << i;
        }
    } else if (S == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) m |= ((int32_t)d[i] > 0 || d[i] > 0xff800000u ? 1u : 0u) << i;
    } else {
        constexpr uint32_t kMinusInf = KEEP == kKeepAboveBF16 ? 0xff80u : 0xfc00u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = d[i] & 0xffffu, hi = d[i] >> 16;
            m |= ((int16_t)lo > 0 || lo > kMinusInf ? 1u : 0u) << (2 * i);
            m |= ((int16_t)hi > 0 || hi > kMinusInf ? 1u : 0u) << (2 * i + 1);
        }
    }
    return m;
}

// out = ReLU(in), bit i of the bitmap set where out[i] is stored by Algorithm 1.  A stream like relu_backward_kernel, a vector a
// lane and 4 KiB a workgroup; G lanes make a bitmap word.  Bound by memory: fp32 8.4 M elements in 11.0 us, where torch.relu and a
// compression without values (which reads that output again and scans it) took 10.9 + 9.9.
template <int S, int KEEP, bool NT>
__global__ __launch_bounds__(kBlock) void relu_forward_kernel(const void *in, const uint64_t n, void *out, uint32_t *__restrict__ bitmap) {
    using G = Geo<S>;
    constexpr int E = G::E;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const uint64_t block_e0 = (uint64_t)blockIdx.x * (kBlock * E), e0 = block_e0 + (uint64_t)threadIdx.x * E;
    const bool full = block_e0 + kBlock * E <= n;
    uint4 v;
    if (full) v = stream_load<NT>(reinterpret_cast<const uint4 *>(static_cast<const char *>(in) + e0 * S));
    else v = load_vec_guarded<S>(in, e0, n);      // (0 beyond n: not kept)
    const uint32_t mk = relu_mask<S, KEEP>(v);
    uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (S == 8) d[j] &= 0u - ((mk >> (j >> 1)) & 1u);
        else if (S == 4) d[j] &= 0u - ((mk >> j) & 1u);
        else d[j] &= (((mk >> (2 * j)) & 1u) * 0x0000ffffu) | (((mk >> (2 * j + 1)) & 1u) * 0xffff0000u);
    }
    const uint4 o = make_uint4(d[0], d[1], d[2], d[3]);
    if (full) stream_store<kReluNtStore>(reinterpret_cast<uint4 *>(static_cast<char *>(out) + e0 * S), o);
    else store_vec_guarded<S>(out, e0, n, o);
    const uint32_t word = group_or<G::G>(mk << (uint32_t)(E * (lane % G::G)));
    if (lane % G::G == 0 && e0 < n) bitmap[e0 >> 5] = word;
}

// ---- small fills ---------------------------------------------------------------------------

__global__ void fill_u64_kernel(uint64_t *p, uint64_t count, uint64_t value) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = value;
}

// Compression of no elements.
__global__ void no_values_kernel(uint64_t *nnz) {
    if (threadIdx.x == 0) store_nnz(nnz, 0);
}

// bt_workspace_status: d_status[0] = 1 if a wait was given up on the workspace (else 0), d_status[1] = calls completed.
__global__ void copy_status_kernel(const uint32_t *ws, uint32_t *d_status) {
    if (threadIdx.x == 0) {
        d_status[0] = ws[kHdrError] != 0 ? 1u : 0u;
        d_status[1] = ws[kHdrCalls];
    }
}

// ---- host side ---------------------------------------------------------------------------------

int elem_size(bt_dtype dt) {
    switch (dt) {
        case BT_F32: return 4;
        case BT_F16: return 2;
        case BT_BF16: return 2;
        case BT_F64: return 8;
    }
    return 0;
}

uint64_t tile_elems(int s, int rows = kRows) { return (uint64_t)kBlock * rows * (kVecBytes / s); }

uint64_t tiles_for(uint64_t n, int s, int rows = kRows) {
    const uint64_t t = tile_elems(s, rows);
    return (n + t - 1) / t;
}

constexpr uint64_t kReluCachedBytes = (uint64_t)48 << 20;      // largest gradient that is read through the caches

// A stream over n elements, `per_block` (a multiple of 32) a workgroup: go(first element, elements, workgroups) for one launch, or
// for several, since a grid holds less than 2^32 threads.
template <class Go> bt_status stream_launches(uint64_t n, uint64_t per_block, Go go) {
    const uint64_t most = per_block << 23;      // 2^31 threads
    for (uint64_t first = 0; first < n; first += most) {
        const uint64_t count = n - first < most ? n - first : most;
        const bt_status st = go(first, count, (count + per_block - 1) / per_block);
        if (st != BT_OK) return st;
    }
    return BT_OK;
}

bool misaligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

// A launch is most of what a small call costs.  hipLaunchKernel itself, whose status is this launch's own: the triple brackets
// go through it too, after putting the configuration aside and taking it up again, and then need hipGetLastError to learn how it
// went (measured 2.45 us a launch, now 2.2).
template <class... P>
bt_status launch(void (*kernel)(P...), uint64_t grid, int block, hipStream_t hs, const std::common_type_t<P> &...args) {
    void *where[] = {const_cast<void *>(static_cast<const void *>(&args))...};
    if (hipLaunchKernel(reinterpret_cast<const void *>(kernel), dim3((unsigned)grid), dim3((unsigned)block), where, 0, hs) == hipSuccess) return BT_OK;
    (void)hipGetLastError();
    return BT_ERR_HIP;
}

constexpr int kMaxDevices = 64;          // devices the static workspace keeps an address for

bt_status check_common(uint64_t n, bt_dtype dt, const void *d_ws, size_t ws_bytes) {
    if (elem_size(dt) == 0) return BT_ERR_DTYPE;
    if (n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
    if (n == 0) return BT_OK;
    if (d_ws == nullptr) return BT_ERR_NULL;
    if (misaligned(d_ws, 128)) return BT_ERR_ALIGN;
    if (ws_bytes < bt_workspace_bytes(n, dt)) return BT_ERR_WORKSPACE;
    return BT_OK;
}

// Slots that a batch's workspace has for a tensor of n elements: its tiles rounded up to whole rows of 128, at least one.
// (Launches take a slot a tile; the size of a workspace is part of the interface.)
uint64_t batch_slots_for(uint64_t n, int s) {
    const uint64_t tiles = tiles_for(n, s);
    return ((tiles == 0 ? 1 : tiles) + 127) / 128 * 128;
}

size_t workspace_bytes_for_slots(uint64_t slots) {
    uint64_t blocks = (slots + kSlotsPerBlock - 1) / kSlotsPerBlock;
    if (blocks == 0) blocks = 1;
    return kHeaderBytes + (size_t)blocks * kBlockBytes;
}

// Tensors [first, first + count) of a batch, laid end to end.  `n_of(i)` is tensor i's element count.
template <int MAXB, class NOf>
void lay_out(BatchLayout<MAXB> &lay, size_t first, size_t count, int s, NOf n_of) {
    lay.count = (uint32_t)count;
    uint64_t at = 0;
    for (size_t i = 0; i < count; ++i) {
        lay.start[i] = (uint32_t)at;
        at += tiles_for(n_of(first + i), s);
    }
    constexpr size_t kStarts = sizeof(lay.start) / sizeof(lay.start[0]);
    for (size_t i = count; i < kStarts; ++i) lay.start[i] = (uint32_t)at;
    for (size_t i = 0; i < 8; ++i) lay.coarse[i] = 8 * i < kStarts ? lay.start[8 * i] : (uint32_t)at;
}

// Largest workspace any launch of the batch needs when it is cut into consecutive launches of `per_launch`
// tensors, which reuse the workspace.
template <class NOf>
size_t batch_workspace_bytes(size_t count, size_t per_launch, int s, NOf n_of) {
    size_t need = workspace_bytes_for_slots(0);
    for (size_t first = 0; first < count; first += per_launch) {
        const size_t c = count - first < per_launch ? count - first : per_launch;
        uint64_t slots = 0;
        for (size_t i = 0; i < c; ++i) slots += batch_slots_for(n_of(first + i), s);
        const size_t b = workspace_bytes_for_slots(slots);
        if (b > need) need = b;
    }
    return need;
}

bt_status check_batch_common(const void *items, size_t count, bt_dtype dt, const void *d_ws) {
    if (elem_size(dt) == 0) return BT_ERR_DTYPE;
    if (count == 0) return BT_OK;
    if (items == nullptr || d_ws == nullptr) return BT_ERR_NULL;
    if (misaligned(d_ws, 128)) return BT_ERR_ALIGN;
    return BT_OK;
}

// Tiles of two rows that one XCD takes by itself, its share of a launch of eight times as many workgroups of which the others end at once.
// XCDs begin a launch up to a microsecond one after the other, and a tile waits for the counts of all before it: with all of
// them on the one that begins first there is nothing to wait for but the counts, as long as one XCD's memory paths do for the tensor.
// Nothing rests on where the workgroups really go.  Measured, us, on all XCDs / on one: fp32 12.5 k elements 3.75 / 3.41, 25 k 3.98 / 3.51, 50 k
// (25 tiles) 3.99 / 3.50, 75 k 4.08 / 3.98, 100 k 4.25 / 4.32; bf16 12.5 k 3.64 / 3.36, 65 k 3.95 / 3.51, 130 k 4.12 / 3.90; fp64 12.5 k 3.97 / 3.44; activation
// calls, which store more, fp32 12.5 k 3.79 / 3.60, 50 k 3.96 / 4.07, fp64 12.5 k 3.88 / 3.97: not done.
constexpr uint64_t kOneXcdSlots = 28;

// Launch the compression kernel for a dtype / pruning / dense-output combination on `job`.
template <int R, int DIRECT, class Job>
bt_status launch_compress(const Job &job, uint64_t slots, bt_dtype dtype, bool prune, bool dense, double threshold,
                          char *ws, hipStream_t hs) {
    static_assert(R != 2 || DIRECT != 0, "tiles of two rows have no scanner");
    // A workspace is sized in tiles of kRows rows (bt_workspace_bytes) and has one block at the least: that one is all that a launch
    // of smaller tiles can count on, whose counts would lie behind the workspace beyond it.
    static_assert(R == kRows || (DIRECT != 0 && DIRECT <= kSlotsPerBlock), "smaller tiles have the slots of one block");
    const uint64_t grid = R == 2 && !dense && slots <= kOneXcdSlots ? slots << kLog2Xcds : slots + (DIRECT ? 0u : 1u);      // with or without a scanner
    // Elements narrower than a double are compared in single precision.  For a single x, x > threshold exactly when
    // x > the largest single at or below the threshold, so that is what the kernel gets (a NaN stays one: nothing
    // exceeds it).
    float threshold_f = (float)threshold;
    if ((double)threshold_f > threshold) threshold_f = std::nextafterf(threshold_f, -INFINITY);
    const auto go = [&](auto kernel) { return launch(kernel, grid, kBlock, hs, job, ws, threshold, threshold_f); };
    const int s = elem_size(dtype);
    // (What compress_common does not launch with four waves waiting is not built either.)
    constexpr bool kQuarters = DIRECT > (int)kDirectSlots;
    if (!prune) {
        if (s == 4) return go(compress_kernel<4, R, DIRECT, kKeepNonZero, false, Job>);
        if (s == 2) return go(compress_kernel<2, R, DIRECT, kKeepNonZero, false, Job>);
        if constexpr (!kQuarters) return go(compress_kernel<8, R, DIRECT, kKeepNonZero, false, Job>);
    } else if (!dense) {
        if (dtype == BT_F32) return go(compress_kernel<4, R, DIRECT, kKeepAboveF32, false, Job>);
        if (dtype == BT_F16) return go(compress_kernel<2, R, DIRECT, kKeepAboveF16, false, Job>);
        if (dtype == BT_BF16) return go(compress_kernel<2, R, DIRECT, kKeepAboveBF16, false, Job>);
        if constexpr (!kQuarters) return go(compress_kernel<8, R, DIRECT, kKeepAboveF64, false, Job>);
    } else {
        if (dtype == BT_F64) return go(compress_kernel<8, R, DIRECT, kKeepAboveF64, true, Job>);
        if (dtype == BT_F32) return go(compress_kernel<4, R, DIRECT, kKeepAboveF32, true, Job>);
        if constexpr (!kQuarters) return go(dtype == BT_F16 ? compress_kernel<2, R, DIRECT, kKeepAboveF16, true, Job> : compress_kernel<2, R, DIRECT, kKeepAboveBF16, true, Job>);
    }
    return BT_ERR_UNSUPPORTED;
}

template <int MODE, class Job> bt_status launch_decompress(const Job &job, uint64_t slots, int s, char *ws, hipStream_t hs) {
    const auto go = [&](auto kernel) { return launch(kernel, slots + (MODE == kQuartered ? 0 : 1), kBlock, hs, job, ws); };      // with or without a scanner
    if (s == 4) return go(decompress_kernel<4, MODE, Job>);
    if (s == 2) return go(decompress_kernel<2, MODE, Job>);
    if constexpr (MODE == kQuartered) return BT_ERR_UNSUPPORTED;      // (bt_decompress has none of these)
    else return go(decompress_kernel<8, MODE, Job>);
}

template <int R, int W> bt_status launch_decompress_small(const DecompressOne &job, uint64_t tiles, int s, char *ws, hipStream_t hs) {
    const auto go = [&](auto kernel) { return launch(kernel, tiles, W * kWaveSize, hs, job, ws); };
    return s == 8 ? go(decompress_small_kernel<8, R, W>) : s == 4 ? go(decompress_small_kernel<4, R, W>) : go(decompress_small_kernel<2, R, W>);
}

template <class Job> bt_status launch_decompress_indexed(const Job &job, uint64_t slots, int s, hipStream_t hs) {
    constexpr uint64_t kMost = 1u << 22;      // slots a launch: a grid holds less than 2^32 threads
    for (uint64_t first = 0; first < slots; first += kMost) {
        const auto go = [&](auto kernel) { return launch(kernel, 2 * (slots - first < kMost ? slots - first : kMost), kBlock, hs, job, (uint32_t)first); };
        const bt_status st = s == 8 ? go(decompress_indexed_kernel<8, Job>) : s == 4 ? go(decompress_indexed_kernel<4, Job>) : go(decompress_indexed_kernel<2, Job>);
        if (st != BT_OK) return st;
    }
    return BT_OK;
}

// ---- a workspace that belongs to the library -------------------------------------------------
//
// For callers that cannot allocate (see bt_compress_static in the header): a workspace for tensors of
// up to BT_STATIC_MAX_TILES tiles, one copy on every device the library is used on, held until the
// process ends.  In host code the array's name only stands for the symbol: what kernels and fills get is
// the address that the runtime reports for it on the current device, looked up once per device.
constexpr size_t kStaticBytes = kHeaderBytes + (size_t)(BT_STATIC_MAX_TILES / kSlotsPerBlock) * kBlockBytes;
static_assert(BT_STATIC_MAX_TILES % kSlotsPerBlock == 0, "whole blocks");
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

bt_status static_workspace(char **ws) {
    static std::atomic<char *> known[kMaxDevices];
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) {
        (void)hipGetLastError();
        return BT_ERR_HIP;
    }
    char *ptr = known[device].load(std::memory_order_acquire);
    if (ptr == nullptr) {
        if (hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) {
            (void)hipGetLastError();
            return BT_ERR_HIP;
        }
        known[device].store(ptr, std::memory_order_release);      // (two threads may both look it up: same answer)
    }
    *ws = ptr;
    return BT_OK;
}

}  // namespace

extern "C" {

size_t bt_dtype_size(bt_dtype dtype) { return (size_t)elem_size(dtype); }

size_t bt_bitmap_bytes(uint64_t n) { return (size_t)(4 * ((n + 31) / 32)); }

size_t bt_compressed_size(uint64_t n, uint64_t nnz, bt_dtype dtype) {
    const int s = elem_size(dtype);
    if (s == 0 || nnz > n) return 0;
    return (size_t)(4 * ((n + 31) / 32) + nnz * (uint64_t)s);
}

size_t bt_dense_size(uint64_t n, bt_dtype dtype) { return (size_t)(n * (uint64_t)elem_size(dtype)); }

size_t bt_coo_size(uint64_t nnz, uint32_t ndim, uint32_t index_bytes, bt_dtype dtype) {
    const int s = elem_size(dtype);
    if (s == 0 || ndim == 0 || (index_bytes != 4 && index_bytes != 8)) return 0;
    return (size_t)(((uint64_t)s + (uint64_t)index_bytes * ndim) * nnz);
}

size_t bt_workspace_bytes(uint64_t n, bt_dtype dtype) {
    const int s = elem_size(dtype);
    if (s == 0) return 0;
    return workspace_bytes_for_slots(tiles_for(n, s));
}

const char *bt_status_str(bt_status status) {
    switch (status) {
        case BT_OK: return "ok";
        case BT_ERR_NULL: return "null pointer";
        case BT_ERR_DTYPE: return "unknown dtype";
        case BT_ERR_ALIGN: return "misaligned pointer";
        case BT_ERR_WORKSPACE: return "workspace too small";
        case BT_ERR_HIP: return "HIP launch failed";
        case BT_ERR_SIZE: return "element count too large";
        case BT_ERR_UNSUPPORTED: return "not available in this build of the library";
    }
    return "unknown status";
}

bt_status bt_workspace_init(void *d_workspace, size_t workspace_bytes, bt_stream stream) {
    if (d_workspace == nullptr) return BT_ERR_NULL;
    if (misaligned(d_workspace, 128)) return BT_ERR_ALIGN;
    const uint64_t count = workspace_bytes / 8;
    if (count == 0) return BT_OK;
    return launch(fill_u64_kernel, (count + 255) / 256, 256, (hipStream_t)stream, (uint64_t *)d_workspace, count, (uint64_t)0);
}

static bt_status compress_common(const void *d_in, uint64_t n, bt_dtype dtype, bool prune, double threshold,
                                 uint32_t *d_bitmap, void *d_values, uint64_t values_cap, uint64_t *d_nnz,
                                 uint64_t *d_index, void *d_dense, void *d_workspace, size_t workspace_bytes,
                                 bt_stream stream) {
    const bt_status st = check_common(n, dtype, d_workspace, workspace_bytes);
    if (st != BT_OK) return st;
    if (d_nnz == nullptr) return BT_ERR_NULL;
    if (misaligned(d_nnz, 8)) return BT_ERR_ALIGN;
    const int s = elem_size(dtype);
    hipStream_t hs = (hipStream_t)stream;
    if (n == 0) {
        return launch(no_values_kernel, 1, 64, hs, d_nnz);
    }
    if (d_in == nullptr || d_bitmap == nullptr) return BT_ERR_NULL;
    if (d_values == nullptr && values_cap != 0) return BT_ERR_NULL;
    if (misaligned(d_in, 16) || misaligned(d_bitmap, 4) || misaligned(d_values, (size_t)s)) return BT_ERR_ALIGN;

    char *const ws = static_cast<char *>(d_workspace);
    const auto go = [&](auto rows, auto direct) {
        constexpr int R = decltype(rows)::value;
        const uint32_t n_tiles = (uint32_t)tiles_for(n, s, R);
        const CompressOne job{d_in, n, d_bitmap, d_values, values_cap, d_nnz, d_index, d_dense, n_tiles};
        return launch_compress<R, decltype(direct)::value>(job, n_tiles, dtype, prune, d_dense != nullptr, threshold, ws, hs);
    };
    // Small tensors.  With few tiles a launch is the chain kernel start, load, count, wait, store, each step at the latency of
    // a wave that has its SIMD nearly to itself, so a tile of two or four rows a lane instead of eight is through sooner,
    // as long as no more than kDirectSlots workgroups poll each other's counts; two rows only up to 64 tiles, beyond which
    // the polling costs more than they save.  An index entry comes from every second or fourth of these tiles.  Measured,
    // us per call on the GPU, before / after: fp32 5 k elements 6.1 / 3.6, 50 k 5.9 / 4.1, 201 k 6.5 / 4.5 (with two rows 4.7), 500 k
    // 6.3 / 4.9, 1 M 6.6 / 5.2, 2 M (eight rows) 7.3 / 6.2; bf16 2 M 7.0 / 5.3.  With an index: bf16 100 k elements
    // with the scanner 7.2, without it but in tiles of eight rows 7.3 (by the workspace's place up to 7.6), of two rows 4.8; 800 k,
    // 5 % zeros, 8.7 / 9.2 / 6.3 (four rows); fp32 201 k 6.9 / 6.6 / 4.8.
    using std::integral_constant;
    const integral_constant<int, (int)kDirectSlots> direct;
    const integral_constant<int, kRows> eight;
    const uint64_t tiles = tiles_for(n, s);
    if (tiles_for(n, s, 2) <= 64) return go(integral_constant<int, 2>{}, direct);
    if (tiles_for(n, s, 4) <= kDirectSlots) return go(integral_constant<int, 4>{}, direct);
    if (tiles <= kDirectSlots) return go(eight, direct);
    // More tiles than that, still without a scanner: all four waves read counts (wait_for_quarter).  Where it stops is where the tiles'
    // polls get into each other's way and into that of the values: with many values sooner, and with a dense output beside them
    // for 16-bit elements at once.  Measured, us, with the scanner / this: fp32 2.2 M elements (269 tiles) 7.3 / 6.7, 3.2 M 8.2 / 7.0, at 95 %
    // zeros 7.8 / 6.5, at 5 % 9.1 / 9.0, 3.9 M 8.5 / 7.7, at 5 % 9.3 / 9.5 (not done), 8 M 11.1 / 15.2; pruning 3.2 M 8.4 / 7.4; activation call 3.2 M 8.4 / 8.2;
    // bf16 4.3 M (263) 7.4 / 7.2, 8.4 M (512) 9.0 / 7.9, at 5 % 9.8 / 8.4, at 95 % 8.3 / 7.3, activation call 4.5 M 9.0 / 9.2; fp64 1.6 M (391) 8.2 / 8.0, at 5 %
    // 8.8 / 9.7, activation call 1.1 M 7.7 / 7.1, 2.1 M (512) 8.9 / 8.1.  The lines hold for pruning and with an index as well, us, at 50 / 5 / 95 %
    // zeros: pruning fp32 3.7 M (448) 8.5 / 7.3, 9.1 / 8.6, 7.9 / 6.8, bf16 4.3 M 7.8 / 7.8, 8.9 / 8.3, -, 8.4 M 9.1 / 8.4, 10.0 / 8.8, 8.3 / 7.6, fp16 8.4 M 9.2 / 8.6,
    // 10.0 / 8.9, 8.5 / 7.8; indexed fp32 3.7 M 8.5 / 7.1, 9.3 / 8.9, 7.8 / 6.5, bf16 8.4 M 8.8 / 7.9, 9.5 / 8.4, 8.1 / 7.1, fp16 8.4 M 8.8 / 7.8, 9.5 / 8.5, -.
    const bool dense = d_dense != nullptr;
    const uint64_t most = s == 4 ? 448 : dense == (s == 8) ? kQuarterSlots : 0;
    if (tiles <= most) return go(eight, integral_constant<int, (int)kQuarterSlots>{});
    return go(eight, integral_constant<int, 0>{});
}

bt_status bt_compress(const void *d_in, uint64_t n, bt_dtype dtype, uint32_t *d_bitmap, void *d_values,
                      uint64_t values_cap, uint64_t *d_nnz, void *d_workspace, size_t workspace_bytes,
                      bt_stream stream) {
    return compress_common(d_in, n, dtype, false, 0.0, d_bitmap, d_values, values_cap, d_nnz, nullptr, nullptr,
                           d_workspace, workspace_bytes, stream);
}

bt_status bt_compress_static(const void *d_in, uint64_t n, bt_dtype dtype, uint32_t *d_bitmap, void *d_values,
                             uint64_t values_cap, uint64_t *d_nnz, bt_stream stream) {
    const int s = elem_size(dtype);
    if (s == 0) return BT_ERR_DTYPE;
    if (n > BT_MAX_ELEMENTS || tiles_for(n, s) > BT_STATIC_MAX_TILES) return BT_ERR_SIZE;
    char *ws = nullptr;
    const bt_status st = static_workspace(&ws);
    if (st != BT_OK) return st;
    // The array keeps what the last call left, possibly a call that gave up a wait: start from a clean workspace
    // every time (a fill kernel rather than a memset, which callers that record the stream could not replay).
    const uint64_t words = kStaticBytes / 8;
    const bt_status fs = launch(fill_u64_kernel, (words + 255) / 256, 256, (hipStream_t)stream, reinterpret_cast<uint64_t *>(ws), words, (uint64_t)0);
    if (fs != BT_OK) return fs;
    return compress_common(d_in, n, dtype, false, 0.0, d_bitmap, d_values, values_cap, d_nnz, nullptr, nullptr, ws,
                           kStaticBytes, stream);
}

bt_status bt_compress_pruned(const void *d_in, uint64_t n, bt_dtype dtype, double threshold, uint32_t *d_bitmap,
                             void *d_values, uint64_t values_cap, uint64_t *d_nnz, void *d_workspace,
                             size_t workspace_bytes, bt_stream stream) {
    return compress_common(d_in, n, dtype, true, threshold, d_bitmap, d_values, values_cap, d_nnz, nullptr, nullptr,
                           d_workspace, workspace_bytes, stream);
}

bt_status bt_activation_compress(const void *d_in, uint64_t n, bt_dtype dtype, double threshold, void *d_dense_out,
                                 uint32_t *d_bitmap, void *d_values, uint64_t values_cap, uint64_t *d_nnz,
                                 void *d_workspace, size_t workspace_bytes, bt_stream stream) {
    if (elem_size(dtype) != 0 && n != 0 && n <= BT_MAX_ELEMENTS) {
        if (d_dense_out == nullptr) return BT_ERR_NULL;
        if (misaligned(d_dense_out, 16)) return BT_ERR_ALIGN;
    }
    return compress_common(d_in, n, dtype, true, threshold, d_bitmap, d_values, values_cap, d_nnz, nullptr, d_dense_out,
                           d_workspace, workspace_bytes, stream);
}

size_t bt_tile_elems(bt_dtype dtype) {
    const int s = elem_size(dtype);
    return s == 0 ? 0 : (size_t)tile_elems(s);
}

size_t bt_index_bytes(uint64_t n, bt_dtype dtype) {
    const int s = elem_size(dtype);
    return s == 0 ? 0 : (size_t)(8 * tiles_for(n, s));
}

bt_status bt_compress_indexed(const void *d_in, uint64_t n, bt_dtype dtype, uint32_t *d_bitmap, void *d_values,
                              uint64_t values_cap, uint64_t *d_nnz, uint64_t *d_index, void *d_workspace,
                              size_t workspace_bytes, bt_stream stream) {
    if (elem_size(dtype) != 0 && n != 0 && n <= BT_MAX_ELEMENTS) {
        if (d_index == nullptr) return BT_ERR_NULL;
        if (misaligned(d_index, 8)) return BT_ERR_ALIGN;
    }
    return compress_common(d_in, n, dtype, false, 0.0, d_bitmap, d_values, values_cap, d_nnz, d_index, nullptr,
                           d_workspace, workspace_bytes, stream);
}

bt_status bt_decompress_indexed(const uint32_t *d_bitmap, const void *d_values, uint64_t values_cap,
                                const uint64_t *d_index, uint64_t n, bt_dtype dtype, void *d_out, bt_stream stream) {
    const int s = elem_size(dtype);
    if (s == 0) return BT_ERR_DTYPE;
    if (n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
    if (n == 0) return BT_OK;
    if (d_bitmap == nullptr || d_out == nullptr || d_index == nullptr) return BT_ERR_NULL;
    if (d_values == nullptr && values_cap != 0) return BT_ERR_NULL;
    if (misaligned(d_out, 16) || misaligned(d_bitmap, 4) || misaligned(d_values, (size_t)s) || misaligned(d_index, 8))
        return BT_ERR_ALIGN;
    const uint32_t n_tiles = (uint32_t)tiles_for(n, s);
    const DecompressOne job{d_bitmap, d_values, values_cap, d_index, n, d_out, n_tiles};
    return launch_decompress_indexed(job, n_tiles, s, (hipStream_t)stream);
}

bt_status bt_decompress(const uint32_t *d_bitmap, const void *d_values, uint64_t n, bt_dtype dtype, void *d_out,
                        void *d_workspace, size_t workspace_bytes, bt_stream stream) {
    const bt_status st = check_common(n, dtype, d_workspace, workspace_bytes);
    if (st != BT_OK) return st;
    if (n == 0) return BT_OK;
    const int s = elem_size(dtype);
    if (d_bitmap == nullptr || d_out == nullptr) return BT_ERR_NULL;   // d_values may be NULL when nnz == 0
    if (misaligned(d_out, 16) || misaligned(d_bitmap, 4) || misaligned(d_values, (size_t)s)) return BT_ERR_ALIGN;
    char *const ws = static_cast<char *>(d_workspace);
    hipStream_t hs = (hipStream_t)stream;
    const auto job = [&](uint64_t tiles) { return DecompressOne{d_bitmap, d_values, ~(uint64_t)0, nullptr, n, d_out, (uint32_t)tiles}; };
    // Small tensors: every workgroup counts the bitmap before its tile itself, in tiles of two rows a lane or, with eight waves, of four
    // (the tiles of the index).  What a workgroup reads grows with the tensor, to the whole bitmap at its end: 256 KiB at 2 M elements, which
    // is where the scanner is as fast (224 KiB for wider elements: at 5 % zeros fp32 2.09 M 6.6 with it, 7.0 without).  Measured, us per call on
    // the GPU, before / after: fp32 5 k elements 6.0 / 2.9, 201 k 6.5 / 3.2, 500 k 6.7 / 3.6.  Two rows up to 320 tiles, against four rows above 256:
    // fp32 560 k 4.4 / 4.1, bf16 1.06 M 5.5 / 5.3, with eight waves 5.9.  Eight waves, against tiles of four rows and four waves up to 256 of them
    // and the scanner beyond: fp32 800 k 4.8 / 4.5, 1.05 M 5.0 / 4.6, 1.3 M 6.2 / 5.1, 1.6 M 6.1 / 5.5, 2.6 M 7.2 / 7.5; bf16 1.6 M 6.4 / 5.7, 2.09 M
    // 7.3 / 6.6, 3.2 M 6.6 / 7.6; fp64 600 k 5.9 / 4.3, 800 k 6.2 / 4.4, 1.2 M 6.8 / 5.6, 1.8 M 7.5 / 7.3, 2.09 M 7.7 / 7.9.  (Sixteen waves: fp32 1.3 M 5.7,
    // fp64 1.2 M 6.7.)
    const uint64_t tiles2 = tiles_for(n, s, 2), tiles = tiles_for(n, s);
    if (tiles2 <= 320) return launch_decompress_small<2, kWaves>(job(tiles2), tiles2, s, ws, hs);
    if (n <= (s == 2 ? 1u << 21 : 7u << 18)) return launch_decompress_small<4, 2 * kWaves>(job(tiles), tiles, s, ws, hs);
    // (see decompress_kernel)
    if (s != 8 && tiles > kDirectSlots && tiles <= kQuarterSlots) return launch_decompress<kQuartered>(job(tiles), tiles, s, ws, hs);
    if (tiles <= 1024) return launch_decompress<kScannedSoon>(job(tiles), tiles, s, ws, hs);
    return launch_decompress<kScanned>(job(tiles), tiles, s, ws, hs);
}

bt_status bt_relu_backward_from_bitmap(const uint32_t *d_bitmap, const void *d_grad_out, uint64_t n, bt_dtype dtype,
                                       void *d_grad_in, bt_stream stream) {
    const int s = elem_size(dtype);
    if (s == 0) return BT_ERR_DTYPE;
    if (n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
    if (n == 0) return BT_OK;
    if (d_bitmap == nullptr || d_grad_out == nullptr || d_grad_in == nullptr) return BT_ERR_NULL;
    if (misaligned(d_grad_out, 16) || misaligned(d_grad_in, 16) || misaligned(d_bitmap, 4)) return BT_ERR_ALIGN;
    hipStream_t hs = (hipStream_t)stream;
    // The gradient was written just before, so while it fits the 256 MB cache beside what else was written since, it is read
    // from there with plain loads; the hint sends them past it.  Measured, us, with the hint / plain, three sets of buffers in
    // turn: fp32 1 M elements 2.8 / 2.3, 2 M 3.9 / 2.7, 5.5 M 9.2 / 7.8, 12 M 17.5 / 15.2, 20 M 27.3 / 23.8, 25.7 M 34.2 / 35.1; bf16 5.5 M
    // 5.3 / 4.3, 25.7 M 18.6 / 16.1, 60 M 39.5 / 41.1.  With eight sets, which push each other out of it: fp32 5.5 M 9.4 / 7.9, 9 M 13.9 /
    // 13.5, 16 M 22.5 / 23.0, 25.7 M 34.4 / 35.2.  In a step (compress, restore, this) fp32 5.5 M 32.4 / 30.7, 12 M 51.3 / 49.7, bf16 32.2 M 66.4 / 68.4.
    const bool cached = n * (uint64_t)s <= kReluCachedBytes;
    const auto go = [&](auto kernel) {
        return stream_launches(n, (uint64_t)kBlock * kReluRows * (kVecBytes / s), [&](uint64_t first, uint64_t count, uint64_t blocks) {
            return launch(kernel, blocks, kBlock, hs, d_bitmap + first / 32, static_cast<const char *>(d_grad_out) + first * s, count,
                          static_cast<char *>(d_grad_in) + first * s);
        });
    };
    if (s == 8) return go(cached ? relu_backward_kernel<8, false> : relu_backward_kernel<8, true>);
    if (s == 4) return go(cached ? relu_backward_kernel<4, false> : relu_backward_kernel<4, true>);
    return go(cached ? relu_backward_kernel<2, false> : relu_backward_kernel<2, true>);
}

bt_status bt_relu_forward(const void *d_in, uint64_t n, bt_dtype dtype, void *d_out, uint32_t *d_bitmap, bt_stream stream) {
    const int s = elem_size(dtype);
    if (s == 0) return BT_ERR_DTYPE;
    if (n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
    if (n == 0) return BT_OK;
    if (d_in == nullptr || d_out == nullptr || d_bitmap == nullptr) return BT_ERR_NULL;
    if (misaligned(d_in, 16) || misaligned(d_out, 16) || misaligned(d_bitmap, 4)) return BT_ERR_ALIGN;
    hipStream_t hs = (hipStream_t)stream;
    const bool cached = n * (uint64_t)s <= kReluCachedBytes;      // written just before, like a gradient
    const auto go = [&](auto kernel) {
        return stream_launches(n, (uint64_t)kBlock * (kVecBytes / s), [&](uint64_t first, uint64_t count, uint64_t blocks) {
            return launch(kernel, blocks, kBlock, hs, static_cast<const char *>(d_in) + first * s, count, static_cast<char *>(d_out) + first * s,
                          d_bitmap + first / 32);
        });
    };
    if (dtype == BT_F64) return go(cached ? relu_forward_kernel<8, kKeepAboveF64, false> : relu_forward_kernel<8, kKeepAboveF64, true>);
    if (dtype == BT_F32) return go(cached ? relu_forward_kernel<4, kKeepAboveF32, false> : relu_forward_kernel<4, kKeepAboveF32, true>);
    if (dtype == BT_F16) return go(cached ? relu_forward_kernel<2, kKeepAboveF16, false> : relu_forward_kernel<2, kKeepAboveF16, true>);
    return go(cached ? relu_forward_kernel<2, kKeepAboveBF16, false> : relu_forward_kernel<2, kKeepAboveBF16, true>);
}

bt_status bt_mask_apply(const uint32_t *d_bitmap, const void *d_in, uint64_t n, bt_dtype dtype, void *d_out,
                        bt_stream stream) {
    return bt_relu_backward_from_bitmap(d_bitmap, d_in, n, dtype, d_out, stream);
}

size_t bt_batch_workspace_bytes(const uint64_t *n, size_t count, bt_dtype dtype) {
    const int s = elem_size(dtype);
    if (s == 0 || (n == nullptr && count != 0)) return 0;
    const auto n_of = [n](size_t i) { return n[i] > BT_MAX_ELEMENTS ? BT_MAX_ELEMENTS : n[i]; };
    const size_t a = batch_workspace_bytes(count, (size_t)kMaxBatchCompress, s, n_of);
    const size_t b = batch_workspace_bytes(count, (size_t)kMaxBatchDecompress, s, n_of);
    return a > b ? a : b;
}

static bt_status compress_batch_common(const bt_compress_item *items, size_t count, bt_dtype dtype, bool prune,
                                       double threshold, void *d_workspace, size_t workspace_bytes, bt_stream stream) {
    const bt_status st = check_batch_common(items, count, dtype, d_workspace);
    if (st != BT_OK || count == 0) return st;
    const int s = elem_size(dtype);
    size_t with_dense = 0, not_empty = 0;
    for (size_t i = 0; i < count; ++i) {
        const bt_compress_item &it = items[i];
        if (it.n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
        if (it.d_nnz == nullptr) return BT_ERR_NULL;
        if (misaligned(it.d_nnz, 8)) return BT_ERR_ALIGN;
        if (it.n == 0) continue;
        ++not_empty;
        if (it.d_in == nullptr || it.d_bitmap == nullptr) return BT_ERR_NULL;
        if (it.d_values == nullptr && it.values_cap != 0) return BT_ERR_NULL;
        if (misaligned(it.d_in, 16) || misaligned(it.d_bitmap, 4) || misaligned(it.d_values, (size_t)s) ||
            misaligned(it.d_index, 8) || misaligned(it.d_dense_out, 16))
            return BT_ERR_ALIGN;
        if (it.d_dense_out != nullptr) ++with_dense;
    }
    // the dense output is a property of the launch: for every tensor that has elements, or for none
    if (with_dense != 0 && (!prune || with_dense != not_empty)) return BT_ERR_NULL;
    const auto n_of = [items](size_t i) { return items[i].n; };
    if (workspace_bytes < batch_workspace_bytes(count, (size_t)kMaxBatchCompress, s, n_of)) return BT_ERR_WORKSPACE;

    hipStream_t hs = (hipStream_t)stream;
    char *ws = static_cast<char *>(d_workspace);
    for (size_t first = 0; first < count; first += kMaxBatchCompress) {
        const size_t c = count - first < (size_t)kMaxBatchCompress ? count - first : (size_t)kMaxBatchCompress;
        CompressMany b;
        lay_out(b.lay, first, c, s, n_of);
        for (size_t i = 0; i < (size_t)kMaxBatchCompress; ++i) {
            const bt_compress_item it =
                i < c ? items[first + i] : bt_compress_item{nullptr, 0, nullptr, nullptr, 0, nullptr, nullptr, nullptr};
            b.in_[i] = it.d_in;
            b.n_[i] = it.n;
            b.bitmap_[i] = it.d_bitmap;
            b.values_[i] = it.d_values;
            b.cap_[i] = it.values_cap;
            b.nnz_[i] = it.d_nnz;
            b.index_[i] = it.n != 0 ? it.d_index : nullptr;
            b.dense_[i] = it.n != 0 ? it.d_dense_out : nullptr;
        }
        const bt_status ls = launch_compress<kRows, false>(b, b.lay.start[c], dtype, prune, with_dense != 0, threshold, ws, hs);
        if (ls != BT_OK) return ls;
    }
    return BT_OK;
}

bt_status bt_compress_batch(const bt_compress_item *items, size_t count, bt_dtype dtype, void *d_workspace,
                            size_t workspace_bytes, bt_stream stream) {
    return compress_batch_common(items, count, dtype, false, 0.0, d_workspace, workspace_bytes, stream);
}

bt_status bt_compress_batch_pruned(const bt_compress_item *items, size_t count, bt_dtype dtype, double threshold,
                                   void *d_workspace, size_t workspace_bytes, bt_stream stream) {
    return compress_batch_common(items, count, dtype, true, threshold, d_workspace, workspace_bytes, stream);
}

bt_status bt_decompress_batch(const bt_decompress_item *items, size_t count, bt_dtype dtype, void *d_workspace,
                              size_t workspace_bytes, bt_stream stream) {
    const bt_status st = check_batch_common(items, count, dtype, d_workspace);
    if (st != BT_OK || count == 0) return st;
    const int s = elem_size(dtype);
    for (size_t i = 0; i < count; ++i) {
        const bt_decompress_item &it = items[i];
        if (it.n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
        if (it.n == 0) continue;
        if (it.d_bitmap == nullptr || it.d_out == nullptr) return BT_ERR_NULL;   // d_values may be NULL when nnz == 0
        if (misaligned(it.d_out, 16) || misaligned(it.d_bitmap, 4) || misaligned(it.d_values, (size_t)s))
            return BT_ERR_ALIGN;
    }
    const auto n_of = [items](size_t i) { return items[i].n; };
    if (workspace_bytes < batch_workspace_bytes(count, (size_t)kMaxBatchDecompress, s, n_of)) return BT_ERR_WORKSPACE;

    hipStream_t hs = (hipStream_t)stream;
    char *ws = static_cast<char *>(d_workspace);
    for (size_t first = 0; first < count; first += kMaxBatchDecompress) {
        const size_t c = count - first < (size_t)kMaxBatchDecompress ? count - first : (size_t)kMaxBatchDecompress;
        DecompressMany b;
        lay_out(b.lay, first, c, s, n_of);
        for (size_t i = 0; i < (size_t)kMaxBatchDecompress; ++i) {
            const bt_decompress_item it = i < c ? items[first + i] : bt_decompress_item{nullptr, nullptr, 0, nullptr, 0, nullptr};
            b.bitmap_[i] = it.d_bitmap;
            b.values_[i] = it.d_values;
            b.cap_[i] = ~(uint64_t)0;
            b.index_[i] = nullptr;
            b.n_[i] = it.n;
            b.out_[i] = it.d_out;
        }
        const bt_status ls = launch_decompress<kScanned>(b, b.lay.start[c], s, ws, hs);
        if (ls != BT_OK) return ls;
    }
    return BT_OK;
}

bt_status bt_decompress_batch_indexed(const bt_decompress_item *items, size_t count, bt_dtype dtype, bt_stream stream) {
    const int s = elem_size(dtype);
    if (s == 0) return BT_ERR_DTYPE;
    if (count == 0) return BT_OK;
    if (items == nullptr) return BT_ERR_NULL;
    for (size_t i = 0; i < count; ++i) {
        const bt_decompress_item &it = items[i];
        if (it.n > BT_MAX_ELEMENTS) return BT_ERR_SIZE;
        if (it.n == 0) continue;
        if (it.d_bitmap == nullptr || it.d_out == nullptr || it.d_index == nullptr) return BT_ERR_NULL;
        if (it.d_values == nullptr && it.values_cap != 0) return BT_ERR_NULL;
        if (misaligned(it.d_out, 16) || misaligned(it.d_bitmap, 4) || misaligned(it.d_values, (size_t)s) || misaligned(it.d_index, 8))
            return BT_ERR_ALIGN;
    }
    const auto n_of = [items](size_t i) { return items[i].n; };
    hipStream_t hs = (hipStream_t)stream;
    for (size_t first = 0; first < count; first += kMaxBatchDecompress) {
        const size_t c = count - first < (size_t)kMaxBatchDecompress ? count - first : (size_t)kMaxBatchDecompress;
        DecompressMany b;
        lay_out(b.lay, first, c, s, n_of);
        for (size_t i = 0; i < (size_t)kMaxBatchDecompress; ++i) {
            const bt_decompress_item it = i < c ? items[first + i] : bt_decompress_item{nullptr, nullptr, 0, nullptr, 0, nullptr};
            b.bitmap_[i] = it.d_bitmap;
            b.values_[i] = it.d_values;
            b.cap_[i] = it.values_cap;
            b.index_[i] = it.d_index;
            b.n_[i] = it.n;
            b.out_[i] = it.d_out;
        }
        const bt_status ls = launch_decompress_indexed(b, b.lay.start[c], s, hs);      // (nothing for empty tensors only)
        if (ls != BT_OK) return ls;
    }
    return BT_OK;
}

// What the kernels leave in a workspace's header when they had to give up, as words a caller can copy back and look
// at without knowing the layout.
bt_status bt_workspace_status(const void *d_workspace, uint32_t *d_status, bt_stream stream) {
    if (d_workspace == nullptr || d_status == nullptr) return BT_ERR_NULL;
    if (misaligned(d_workspace, 128) || misaligned(d_status, 4)) return BT_ERR_ALIGN;
    return launch(copy_status_kernel, 1, 64, (hipStream_t)stream, static_cast<const uint32_t *>(d_workspace), d_status);
}

}  // extern "C"
