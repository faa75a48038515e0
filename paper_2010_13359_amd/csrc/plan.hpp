// Plan object and internal launchers of the DQGAN library (host side).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <vector>

#include "../../include/dqgan.h"

namespace dq {

// A contiguous run of one segment of a row, at most piece_elems() long; the
// statistics pass reduces one piece per workgroup.  Pieces never cross
// segments.
struct Piece {
    int64_t start;
    int32_t len;
    int32_t seg;
};
// 32768 elements from 16384 workgroups up: the statistics pass over 32 workers
// x 2^25 elements ran 1.5 % faster with them than with 16384, over 16 workers
// x 6.3M elements 2 % slower.  Below kPieceBlocksSmall, four elements less than
// 16384, so that a piece that does not start at a quad takes no trip of its
// own for one quad (8 x 10^6 signs 40.3 -> 39.8 us).
constexpr int64_t kPieceBlocksForLong = 16384, kPieceBlocksSmall = 2048;
inline int64_t piece_elems(int64_t M, int64_t d) {
    if (M * (d / 32768) >= kPieceBlocksForLong) return 32768;
    return M * (d / 16384) >= kPieceBlocksSmall ? 16384 : 16380;
}

// Per (worker, segment) constants of the segment-scaled compressors.
// SIGN: a = the scale.  QSGD, MBIT (equation qsgd): a = fl(s / (u sigma))
// and b = fl(u sigma / s), where u = 2^64 for sigma < 2^-64 (so that s / sigma
// cannot overflow binary32 and sigma / s keeps its significand) and u = 1
// otherwise; with u = 2^64 both are stored negated, and the kernels then
// multiply |p| by 2^64 before the product with |a| and the decoded magnitude
// fl(level * |b|) by 2^-64.  A norm of 0 or one that is not finite gives
// a = b = 0: level 0 everywhere.
struct alignas(8) SegConst {
    float a, b;
};

// Capacity of the MI355X Infinity Cache (memory-side, in front of HBM): the
// fused pass streams message planes larger than this past the caches.
constexpr double kInfinityCacheBytes = 256.0 * 1024 * 1024;

// The first pass of a step (statistics, top-k counts) reads g and e with
// ordinary loads where the Infinity Cache holds them until the second pass has
// read them again; the second does so too where the cache also holds what it
// writes, and the next steps' data.  Otherwise loads stream past the caches
// (with ordinary loads 32 workers x 2^25, s = 15, take 4790 us instead of
// 4490).  What else goes through the cache counts with a weight: w and q-hat,
// which the second pass reads and writes, and the message planes that it
// writes by ordinary stores.  By the size of g and e alone, as measured on
// 4-bit codes of many workers, other steps were up to 17 % slower than with
// streaming loads.
//
// Whole steps over three states in turn: the first pass's ordinary loads stop
// paying at a g and e of about 50 MB with one worker, 95 with two, 143 with
// four, 200 with eight, 250 with sixteen, 285 with 32 (signs, 4-bit codes,
// top-k), and of 117, 145, 178 and 202 MB with 4, 8, 16 and 32 workers, s = 255:
// within 4 % of g + e + 5 (w + q-hat) + 4 planes = 320 MB.  Below the line
// both passes streaming / the first ordinary: 16 workers of 140 MB 81.6 / 76.7
// us, 17 of 187 MB 112.6 / 103.6; above it: 4 workers, s = 255, of 160 MB 97 /
// 107, 8 of 235 MB 138 / 150.  With eight states in turn (nothing left of the
// step before) the line lies lower, at three quarters of that with 4 to 16
// workers; between the two the loss is at most 6 %.
//
// Both passes' ordinary loads stop paying at 50 MB with one worker, 58 with
// two, 72 with four, 83 with eight, 90 with sixteen, 95 with 32, and of the
// identity, whose plane is as large as e, at about 55: g + e + w + q-hat + 2
// planes = 100 MB.  The first ordinary / both: 8 workers, signs, of 60 MB
// 39.0 / 35.9 us; above the line 4 workers, s = 255, of 85 MB 54.5 / 61.0, 8
// workers, identity, of 82 MB 35.4 / 41.5.
constexpr double kFirstPassCached = 320e6, kBothPassesCached = 100e6;
inline double data_bytes(const dqgan_desc &D) { return 8.0 * D.M * static_cast<double>(D.ld); }
inline double vector_bytes(const dqgan_desc &D) { return 8.0 * static_cast<double>(D.ld); }  // w and q-hat
inline double plane_bytes(const dqgan_desc &D) {  // of those written by ordinary stores
    const double n = D.M * static_cast<double>(D.ld);
    switch (D.kind) {
        case DQGAN_SIGN: return n / 8;
        case DQGAN_QSGD: return D.levels == 255 ? n * 9 / 8 : n / 8;
        case DQGAN_MBIT: return D.levels == 8 ? n : 0.0;
        case DQGAN_IDENTITY: return n * 4;
        default: return 0.0;
    }
}
inline bool first_streams(const dqgan_desc &D) {
    return data_bytes(D) + 5 * vector_bytes(D) + 4 * plane_bytes(D) > kFirstPassCached;
}
inline bool second_streams(const dqgan_desc &D) {
    return data_bytes(D) + vector_bytes(D) + 2 * plane_bytes(D) > kBothPassesCached;
}

// The worker's own calls (encode, update) touch the rows once more each: 20 MB
// ordinary / streaming 32.5 / 34.0 us for a worker's iteration, 60 MB 67.0 / 65.5,
// 64 MB 71.9 / 69.3 (s = 255).  The identity has no statistics: its encode is the
// first pass and its update the second, with no plane read in between (one
// worker 120 MB 97.0 / 104.4, 160 MB 133.9 / 138.9, 200 MB 173 / 173, 224 MB 201
// / 193; two 200 MB 0.93 of streaming, 230 0.97; four 230 MB 0.96; sixteen 230 MB
// 0.92).
constexpr double kWorkerCached = 40e6, kWorkerIdentityCached = 275e6;
inline bool worker_streams(const dqgan_desc &D) {
    return D.kind == DQGAN_IDENTITY ? data_bytes(D) + vector_bytes(D) / 2 > kWorkerIdentityCached
                                    : data_bytes(D) > kWorkerCached;
}

// f(STREAM) with `streams` as a compile-time constant.
template <typename F>
void with_stream(bool streams, F &&f) {
    if (streams)
        f(std::true_type{});
    else
        f(std::false_type{});
}

// Per-worker selection state of the top-k compressor.  Keys are the binary32
// bit patterns of |p| (monotone in |p|).  Element i is selected iff
// key > T, or key == T and i <= I.
struct TopkRow {
    uint32_t lo, hi;     // candidate band [lo, hi] of keys, from the sample
    uint32_t n_cand;     // candidates staged into the row's list by the full pass (may exceed the capacity);
                         // this and n_spill, n_above are counted in TopkScratch::ctr and copied here
    uint32_t fallback;   // 1: the band missed the k-th key; the full-row search decides
    uint32_t T, I;       // the selection
    uint32_t n_spill;    // candidates a wave could not stage: stored from the top of the row's list down
    uint32_t total;      // selected count found by the tile scan (equals k)
    uint32_t n_above;    // keys above the band, counted by the full pass
    uint32_t pad[7];
};

constexpr int kTopkTile = 256;            // elements per counting tile (one wave of quads)
// The counters that many workgroups of one kernel update atomically live in
// their own block of TopkScratch::ctr, not in the row's TopkRow: every
// workgroup of the full pass reads its row's band from rows[m] when it
// starts, and the other workgroups' atomics on the same cache line held the
// pass 0.3 ms back at 64 rows of 10^8.  The first search kernel copies the
// pass's counters into rows[m]; the finish reads the play count here.
constexpr int kRowCtrWords = 64;          // words per row (one 256-byte block)
constexpr int kCtrCand = 0, kCtrAbove = 1, kCtrSpill = 2;
constexpr int kCtrPlay = 3;  // candidates still in play after the first key digit, listed for the finish
constexpr int kCtrClaim = 8;      // + phase: chunks of the full-row search claimed by workgroups
constexpr int kCtrFinished = 16;  // + phase: chunks they have finished
constexpr int kTopkChunkTiles = 64;       // tiles per workgroup of the full pass: one candidate run each
constexpr int kSampleBins = 32768;        // sample histogram: key >> 16 (keys < 2^31)
constexpr int kDigitBins = 2048;          // radix-select histograms: 11-bit digits
constexpr int kSelectPasses = 6;          // histogram slots of a search: up to 3 key digits, 3 index digits

// Top-k workspace (one set per plan).
struct TopkScratch {
    TopkRow *rows = nullptr;        // [M]
    uint32_t *ctr = nullptr;        // [M][kRowCtrWords] the full pass's counters of each row, apart from rows
    uint32_t *hist = nullptr;       // [M][kSampleBins] first digit of the sample (zero between iterations); holds
                                    // ref_hist, coarse and done too
    uint32_t *sel_hist = nullptr;   // [M][kDigitBins] histogram of the first key digit among the candidates
    uint2 *play = nullptr;          // [M][cap] the candidates in play after the first key digit
    uint32_t *fb_hist = nullptr;    // [M][kSelectPasses][kDigitBins] digit histograms of the full-row search
    uint2 *cand = nullptr;          // [M][cap] (key, index) candidates: runs from the bottom, spills from the top
    int64_t cap = 0;
    uint2 *runs = nullptr;          // [M][n_chunks] (first position, count) of each full-pass workgroup's candidates
    uint16_t *tile_cnt = nullptr;   // [M][n_tiles] selected elements per 256-element tile (at most 256)
    uint16_t *tile_off = nullptr;   // [M][n_tiles] selected elements before the tile within its chunk (< 2^14)
    uint32_t *chunk_sum = nullptr;  // [M][n_chunks] selected elements per chunk of kTopkChunkTiles tiles
    uint32_t *chunk_off = nullptr;  // [M][n_chunks] exclusive prefix of chunk_sum
    uint32_t *agg_start = nullptr;  // [n_agg_tiles + 1][M] first message entry per server-average tile
    int64_t n_agg_tiles = 0;
    int64_t n_tiles = 0;
    int64_t n_chunks = 0;           // chunks of kTopkChunkTiles tiles per row
    int64_t sample_stride = 0;      // elements from one sampled run to the next
    int64_t n_sample_quads = 0;     // sampled quads per row
    uint32_t *sample_keys = nullptr;  // [M][n_sample_quads][4] the sampled keys of longer rows
    bool row_search = false;        // one workgroup per row searches and scans (k_topk_select_row)
    uint32_t *ref_hist = nullptr;   // [M][2][kDigitBins] second digit of the sample (zero between iterations)
    uint32_t *coarse = nullptr;     // [M][4] first digits of the sample's band (find_bins)
    uint32_t *done = nullptr;       // [M] sample workgroups that have arrived (zero between launches)
    uint32_t n_samples = 0;         // sampled elements per row
};

// The state the apply pass reads: the threshold per row and each tile's
// first output position, tile_off + chunk_off of its chunk.
struct TopkArgs {
    const TopkRow *rows;
    const uint16_t *tile_off;
    const uint32_t *chunk_off;
    int64_t n_tiles;
    int64_t n_chunks;
    int64_t k;
    uint32_t *idx;
};

__device__ __forceinline__ uint32_t topk_tile_base(const TopkArgs &ta, int m, int64_t tile) {
    return ta.tile_off[static_cast<int64_t>(m) * ta.n_tiles + tile] +
           ta.chunk_off[static_cast<int64_t>(m) * ta.n_chunks + tile / kTopkChunkTiles];
}

}  // namespace dq

struct dqgan_plan_s {
    dqgan_desc desc{};
    std::vector<int64_t> offsets;  // host copy, n_seg + 1
    int device = 0;
    int level_bits = 0;            // QSGD: 8 (s = 255) or 4 (s = 15); MBIT: m
    int level_count = 0;           // quantizer levels: QSGD s; MBIT k = 2^(m-1) - 1
    int64_t n_tiles = 0;           // ld / 1024

    int64_t *d_off = nullptr;       // [n_seg + 1]
    int32_t *d_tile_seg = nullptr;  // [n_tiles] segment of each tile's first element
    int32_t max_tile_segs = 1;      // most segments that meet one tile (1024 elements)
    dq::Piece *d_pieces = nullptr;  // [n_pieces]
    int32_t n_pieces = 0;
    int32_t max_seg_pieces = 0;     // most pieces of one segment
    int32_t *d_seg_piece = nullptr;  // [n_seg + 1] first piece of each segment
    double *d_partial = nullptr;     // [M][n_pieces] partial sums (L1, L2^2)
    float *d_pmax = nullptr;         // [M][n_pieces] partial maxima (Linf)
    dq::SegConst *d_consts = nullptr;  // [M][n_seg] per-segment constants
    dq::TopkScratch topk;
};

namespace dq {

// Arrivals of the statistics pass per (worker, segment): in the partials' array
// that the plan's norm leaves unused (each segment has at least one piece).
inline uint32_t *arrivals(const dqgan_plan_s &P) {
    return P.desc.norm == DQGAN_LINF ? reinterpret_cast<uint32_t *>(P.d_partial) : reinterpret_cast<uint32_t *>(P.d_pmax);
}

}  // namespace dq

namespace dq {

// Dense compressors (SIGN, QSGD, MBIT, IDENTITY).
hipError_t launch_segment_scales(const dqgan_plan_s &P, float eta, const float *G, const float *E,
                                 const float *scales_in, float *scale_out, hipStream_t st);
hipError_t launch_consts_from_scales(const dqgan_plan_s &P, const float *scales, hipStream_t st);
hipError_t launch_encode(const dqgan_plan_s &P, float eta, uint32_t t, const float *G, float *E,
                         const dqgan_wire &w, hipStream_t st);
hipError_t launch_fused_dense(const dqgan_plan_s &P, float eta, uint32_t t, const float *G, float *E, float *W,
                              float *WX, const dqgan_wire &w, float *Qhat, hipStream_t st);
hipError_t launch_pack(const dqgan_plan_s &P, const uint16_t *codes, const float *scales, const dqgan_wire &w,
                       hipStream_t st);
hipError_t launch_unpack_dense(const dqgan_plan_s &P, const dqgan_wire &w, float *Phat, hipStream_t st);
hipError_t launch_aggregate_dense(const dqgan_plan_s &P, const dqgan_wire &w, float *Qhat, hipStream_t st);
hipError_t launch_omd(const dqgan_plan_s &P, float eta, const float *Qhat, float *W, const float *G,
                      const float *E, float *WX, hipStream_t st);

// Top-k.
hipError_t topk_alloc(dqgan_plan_s &P);
void topk_free(dqgan_plan_s &P);
hipError_t launch_topk_compress(const dqgan_plan_s &P, float eta, const float *G, float *E, const dqgan_wire &w,
                                hipStream_t st);
hipError_t launch_topk_select(const dqgan_plan_s &P, float eta, const float *G, const float *E, hipStream_t st);
hipError_t launch_topk_apply(const dqgan_plan_s &P, float eta, const float *G, float *E, float *W, float *WX,
                             const dqgan_wire &w, float *Qhat, hipStream_t st);
hipError_t launch_topk_encode_rows(const dqgan_plan_s &P, float eta, const float *G, float *E, const dqgan_wire &w,
                                   hipStream_t st);
hipError_t launch_topk_unpack(const dqgan_plan_s &P, const dqgan_wire &w, float *Phat, hipStream_t st);
hipError_t launch_topk_aggregate(const dqgan_plan_s &P, const dqgan_wire &w, float *Qhat, hipStream_t st);

}  // namespace dq
