// Element-major kernels of Algorithm 2 (arXiv:2010.13359): the statistics
// pass of the segment-scaled compressors (scaled sign, s-level quantizer,
// m-bit sign-magnitude quantizer), the fused apply pass of every compressor
// (top-k included), and the separate pack / unpack / aggregate / OMD kernels.
//
// Passes over HBM per iteration:
//   1. segment statistics: per (worker, segment) sum |p|, sum p^2 or max |p|
//      of p = fl(fl(eta g) + e), one workgroup per piece, binary64 partials;
//      a tiny kernel, or the last workgroup of a segment with few pieces,
//      combines the partials of each segment in piece order (deterministic)
//      into the scale and the quantizer constants.
//   2. the fused apply pass (k_fused_split): a workgroup covers 256 elements
//      of all M workers, its waves splitting the workers; each lane encodes
//      one quad of 4 elements per worker row, writes e_t and the message,
//      keeps p-hat and fl(eta g) + e_t in registers; the ascending-worker sum
//      is chained through LDS; the last wave of the chain applies
//      w_t = w_{t-1} - q-hat; every wave then writes its rows' evaluation
//      points w_t - (fl(eta g) + e_t).  k_fused (one lane walks all M rows)
//      serves M > 256.
#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "plan.hpp"

namespace dq {

namespace {

enum { kSign = DQGAN_SIGN, kQsgd = DQGAN_QSGD, kTopk = DQGAN_TOPK, kIdentity = DQGAN_IDENTITY, kMbit = DQGAN_MBIT };

template <int V>
using Const = std::integral_constant<int, V>;

// How the fused pass treats the caches: its matrices read through them (see
// second_streams), streamed past them, or streamed together with the message.
enum { kIoCached, kIoStream, kIoStreamAll };

// ---------------------------------------------------------------------------
// Pass 1: segment statistics.

// The per-segment constants (SegConst) of a scale: SIGN the scale; QSGD, MBIT
// fl(s/(u sigma)) and fl(u sigma/s), negated when u = 2^64 (sigma < 2^-64),
// zeros for sigma = 0 or not finite.  Quotients of two binary32 values
// computed in binary64 and rounded to binary32 equal the correctly rounded
// binary32 quotient (53 >= 2*24 + 2).
__device__ __forceinline__ SegConst seg_const(int kind, int levels, float sc) {
    SegConst c{sc, 0.0f};
    if (kind == kQsgd || kind == kMbit) {
        c.a = 0.0f;
        if (sc > 0.0f && sc <= 3.402823466e38f) {
            const bool tiny = sc < 0x1.0p-64f;
            // u * sigma is exact: a power of two times a binary32 value
            const double sd = static_cast<double>(sc) * (tiny ? 0x1.0p64 : 1.0), lv = static_cast<double>(levels);
            c.a = static_cast<float>(lv / sd);
            c.b = static_cast<float>(sd / lv);
            if (tiny) {
                c.a = -c.a;
                c.b = -c.b;
            }
        }
    }
    return c;
}

// The scale from the whole segment's sum or maximum; n = its elements.
__device__ __forceinline__ float scale_of(int norm, double s, float mx, int64_t n) {
    return norm == DQGAN_LINF ? mx
           : norm == DQGAN_L1 ? static_cast<float>(s / static_cast<double>(n))
                              : static_cast<float>(sqrt(s));
}

// The scale of one (worker, segment) from its pieces' partials, by a whole
// wave: lane l adds the segment's pieces p0 + l, p0 + l + 64, ... in order,
// then a fixed butterfly combines the lanes (every lane gets the result).
// `partial` and `pmax` point at the worker's row and are read at device scope
// (the statistics pass may have written them in the same launch).
__device__ __forceinline__ float segment_scale(int norm, const double *partial, const float *pmax, int p0, int p1,
                                               int64_t n) {
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    float mx = 0.0f;
    if (norm == DQGAN_LINF) {
        for (int p = p0 + lane; p < p1; p += 64)
            mx = fmaxf(mx, __hip_atomic_load(pmax + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    } else {
        for (int p = p0 + lane; p < p1; p += 64)
            s += __hip_atomic_load(partial + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    }
    return scale_of(norm, s, mx, n);
}

// What the statistics pass writes.
struct StatsOut {
    double *partial;  // [M][n_pieces] per piece
    float *pmax;
    // FEW: [M][n_seg] workgroups of the segment that have arrived (zero between
    // launches)
    uint32_t *arrived;
    const int32_t *seg_piece;
    const int64_t *off;
    float *scale;
    SegConst *consts;
    int32_t n_seg, kind, norm, levels;
};

// FEW: the last workgroup of a segment derives its scale (stats_few); else
// k_finalize does.  A variant of its own: pieces of 100 elements are all head
// and tail, and with the choice made at run time 16 workers x 4M elements in
// such segments took 574 us instead of 506.
template <int NORM, bool STREAM, bool FEW>
__global__ __launch_bounds__(kBlock) void k_segment_partials(const float *__restrict__ G, const float *__restrict__ E,
                                                             float eta, int64_t ld, const Piece *__restrict__ pieces,
                                                             int32_t n_pieces, StatsOut out) {
    const int pc = blockIdx.x;
    const int m = blockIdx.y;
    const Piece P = pieces[pc];
    const float *g = G + static_cast<int64_t>(m) * ld;
    const float *e = E + static_cast<int64_t>(m) * ld;
    const int64_t lo = P.start, hi = P.start + P.len;
    const int64_t q0 = lo >> 2, q1 = (hi + 3) >> 2;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    float mx = 0.0f;
    // Four quads per thread per trip, all eight loads issued before use.
    constexpr int U = 4;
    for (int64_t qb = q0 + threadIdx.x; qb < q1; qb += U * kBlock) {
        f32x4 gv[U], ev[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = qb + u * kBlock;
            if (q < q1) {
                gv[u] = ld_io<STREAM>(g + 4 * q);
                ev[u] = ld_io<STREAM>(e + 4 * q);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = qb + u * kBlock;
            if (q >= q1) break;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t i = 4 * q + c;
                const float p = add_rn(mul_rn(eta, elem(gv[u], c)), elem(ev[u], c));
                const bool in = (i >= lo) && (i < hi);
                if (NORM == DQGAN_L1) {
                    acc[c] += in ? static_cast<double>(fabsf(p)) : 0.0;
                } else if (NORM == DQGAN_L2) {
                    const double pd = static_cast<double>(p);
                    acc[c] += in ? pd * pd : 0.0;  // the product is exact in binary64
                } else {
                    mx = in ? fmaxf(mx, fabsf(p)) : mx;
                }
            }
        }
    }
    __shared__ double sh[kBlock / 64];
    __shared__ float shm[kBlock / 64];
    double s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o);
        mx = fmaxf(mx, __shfl_xor(mx, o));
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[wave] = s;
        shm[wave] = mx;
    }
    __syncthreads();
    const int64_t row = static_cast<int64_t>(m) * n_pieces;
    if constexpr (!FEW) {
        if (threadIdx.x == 0) {
            out.partial[row + pc] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
            out.pmax[row + pc] = fmaxf(fmaxf(shm[0], shm[1]), fmaxf(shm[2], shm[3]));
        }
        return;
    }
    if (wave != 0) return;
    s = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    mx = fmaxf(fmaxf(shm[0], shm[1]), fmaxf(shm[2], shm[3]));
    // Few pieces: the last workgroup of the segment to arrive derives its
    // scale, in place of a launch of its own.
    const int64_t ms = static_cast<int64_t>(m) * out.n_seg + P.seg;
    const int p0 = out.seg_piece[P.seg], p1 = out.seg_piece[P.seg + 1];
    const int64_t n = out.off[P.seg + 1] - out.off[P.seg];
    if (p1 - p0 > 1) {
        // The partial goes out at device scope, the wait holds the arrival
        // back until it is there, and the last to arrive reads all of them at
        // device scope: no cache is written back or dropped, which an
        // agent-scope fence does over the XCD's whole L2.
        uint32_t before = 0;
        if (threadIdx.x == 0) {
            if (NORM == DQGAN_LINF)
                __hip_atomic_store(out.pmax + row + pc, mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else
                __hip_atomic_store(out.partial + row + pc, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            before = __hip_atomic_fetch_add(out.arrived + ms, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (__builtin_amdgcn_readfirstlane(static_cast<int>(before)) != p1 - p0 - 1) return;
        asm volatile("" ::: "memory");
        if (threadIdx.x == 0)  // zero again for the next launch
            __hip_atomic_store(out.arrived + ms, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const float sc = p1 - p0 > 1 ? segment_scale(out.norm, out.partial + row, out.pmax + row, p0, p1, n)
                                 : scale_of(out.norm, s, mx, n);
    if (threadIdx.x != 0) return;
    out.scale[ms] = sc;
    out.consts[ms] = seg_const(out.kind, out.levels, sc);
}

// The scale and constants of every (worker, segment), one wave each, from
// the partials or from the caller's scales.
__global__ __launch_bounds__(kBlock) void k_finalize(int kind, int norm, int levels, const double *__restrict__ partial,
                                                     const float *__restrict__ pmax, int32_t n_pieces,
                                                     const int32_t *__restrict__ seg_piece,
                                                     const int64_t *__restrict__ off, int32_t M, int32_t n_seg,
                                                     const float *__restrict__ scales_in, float *__restrict__ scale_out,
                                                     SegConst *__restrict__ consts) {
    const int64_t tid = (static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x) >> 6;
    if (tid >= static_cast<int64_t>(M) * n_seg) return;
    const int m = static_cast<int>(tid / n_seg);
    const int j = static_cast<int>(tid % n_seg);
    const int64_t row = static_cast<int64_t>(m) * n_pieces;
    const float sc = scales_in ? scales_in[tid]
                               : segment_scale(norm, partial + row, pmax + row, seg_piece[j], seg_piece[j + 1],
                                               off[j + 1] - off[j]);
    if ((threadIdx.x & 63) != 0) return;
    if (scale_out) scale_out[tid] = sc;
    consts[tid] = seg_const(kind, levels, sc);
}

// r = fl(|p| s / sigma) of equation (qsgd) from the constant a of SegConst
// (negative: |p| is first multiplied by 2^64), and the decoded magnitude
// fl(level sigma / s) from its constant b (negative: multiplied back by
// 2^-64).  The extra products are exact or the one final rounding.
__device__ __forceinline__ float level_ratio(float abs_p, float ca) {
    return mul_rn(mul_rn(abs_p, ca < 0.0f ? 0x1.0p64f : 1.0f), fabsf(ca));
}
__device__ __forceinline__ float level_magnitude(uint32_t level, float cb) {
    return mul_rn(mul_rn(static_cast<float>(level), fabsf(cb)), cb < 0.0f ? 0x1.0p-64f : 1.0f);
}

// ---------------------------------------------------------------------------
// Per-quad encode of one worker row (shared by the row kernel and the fused
// step).  Outputs: eg = fl(eta g), p-hat, e_t = fl(p - p-hat), the 4 sign bits
// and the 4 level fields (8 bits each, packed low to high).

struct QuadCodes {
    f32x4 eg, phat, enew;
    uint32_t sign_nib;
    uint32_t levels;
};

template <int KIND>
__device__ __forceinline__ QuadCodes encode_quad(const f32x4 g, const f32x4 e, float eta, int64_t i0, int64_t d, int m,
                                                 const int js[4], const SegConst *__restrict__ crow, int s,
                                                 uint32_t k0, uint32_t k1, uint32_t t) {
    QuadCodes o;
    o.sign_nib = 0u;
    o.levels = 0u;
    u32x4 rnd;
    if (KIND == kQsgd || KIND == kMbit) {
        const uint64_t blk = static_cast<uint64_t>(i0) >> 2;
        rnd = philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(m), t, static_cast<uint32_t>(blk >> 32),
                            k0, k1);
    }
    const float fs = static_cast<float>(s);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float gc = elem(g, c), ec = elem(e, c);
        const float egc = mul_rn(eta, gc);
        const float p = add_rn(egc, ec);
        float q = 0.0f, en = ec, egk = 0.0f;
        uint32_t neg = 0u, level = 0u;
        if (i0 + c < d) {
            egk = egc;
            neg = signbit(p) ? 1u : 0u;
            if (KIND == kSign) {
                const float sc = crow[js[c]].a;
                q = neg ? -sc : sc;
            } else if (KIND == kQsgd || KIND == kMbit) {
                const SegConst cs = crow[js[c]];
                const float a = fabsf(p);
                if (cs.a != 0.0f && a > 0.0f) {
                    const float r = level_ratio(a, cs.a);
                    const float l = fminf(floorf(r), fs);
                    const float frac = (l == fs) ? 0.0f : sub_rn(r, l);
                    const float u = static_cast<float>(elem(rnd, c) >> 8) * 0x1.0p-24f;
                    int lv = static_cast<int>(l) + ((u < frac) ? 1 : 0);
                    lv = lv > s ? s : lv;
                    level = static_cast<uint32_t>(lv);
                }
                q = copysignf(level_magnitude(level, cs.b), p);
            } else {
                q = p;
            }
            en = sub_rn(p, q);
        }
        set_elem(o.eg, c, egk);
        set_elem(o.phat, c, q);
        set_elem(o.enew, c, en);
        o.sign_nib |= neg << c;
        o.levels |= level << (8 * c);
    }
    return o;
}

// Top-k (Theorem 1): p-hat = p on the selected elements, 0 elsewhere;
// sign_nib carries the selection mask of the quad.
__device__ __forceinline__ QuadCodes encode_quad_topk(const f32x4 g, const f32x4 e, float eta, int64_t i0, int64_t d,
                                                      uint32_t T, uint32_t I) {
    QuadCodes o;
    o.sign_nib = 0u;
    o.levels = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float gc = elem(g, c), ec = elem(e, c);
        const float egc = mul_rn(eta, gc);
        const float p = add_rn(egc, ec);
        float q = 0.0f, en = ec, egk = 0.0f;
        const int64_t i = i0 + c;
        if (i < d) {
            egk = egc;
            const uint32_t key = __float_as_uint(p) & 0x7FFFFFFFu;
            const bool sel = key > T || (key == T && static_cast<uint32_t>(i) <= I);
            q = sel ? p : 0.0f;
            en = sub_rn(p, q);
            o.sign_nib |= (sel ? 1u : 0u) << c;
        }
        set_elem(o.eg, c, egk);
        set_elem(o.phat, c, q);
        set_elem(o.enew, c, en);
    }
    return o;
}

// Ordered compaction of one row's selected elements of a 256-element tile
// (the wave's 64 quads, element 4*lane + c): the position is the tile's
// offset plus the number of selected elements before it in the tile.
__device__ __forceinline__ void store_topk(float *__restrict__ val_row, uint32_t *__restrict__ idx_row, int64_t k,
                                           uint32_t tile_base, int64_t i0, const QuadCodes &cq) {
    const uint32_t mask = cq.sign_nib;
    const int lane = threadIdx.x & 63;
    const uint64_t below = (uint64_t(1) << lane) - 1;
    uint32_t pre = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) pre += __popcll(__ballot((mask >> c) & 1u) & below);
    // Store round r writes each lane's r-th selected element: at a low
    // selection density almost every wave needs one round (two store
    // instructions) instead of one per element position of the quad.
    const uint32_t n_sel = __popc(mask);
    uint32_t rest = mask;
    for (uint32_t r = 0; __ballot(r < n_sel) != 0; ++r) {
        if (r < n_sel) {
            const int c = __ffs(rest) - 1;
            rest &= rest - 1;
            const int64_t pos = static_cast<int64_t>(tile_base) + pre + r;
            if (pos < k) {
                val_row[pos] = elem(cq.phat, c);
                idx_row[pos] = static_cast<uint32_t>(i0 + c);
            }
        }
    }
}

// The segments of the quad at i0 (elements at or beyond d: the last one's), from
// a segment j that does not lie behind them.
__device__ __forceinline__ void walk_segments(const int64_t *__restrict__ off, int j, int64_t i0, int64_t d,
                                              int js[4]) {
    const int64_t last = d - 1;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int64_t i = i0 + c;
        j = seg_from(off, j, i < last ? i : last);
        js[c] = j;
    }
}
__device__ __forceinline__ void lookup_segments(const int64_t *__restrict__ off, const int32_t *__restrict__ tile_seg,
                                                int64_t i0, int64_t d, int js[4]) {
    walk_segments(off, tile_seg[i0 >> 10], i0, d, js);
}

// The segment of element min(i, d - 1), for an i that is the same for the
// whole wave: scalar loads, off the vector memory queue.
__device__ __forceinline__ int uniform_segment(const int64_t *__restrict__ off, const int32_t *__restrict__ tile_seg,
                                               int64_t i, int64_t d) {
    return seg_from(off, tile_seg[i >> 10], i < d ? i : d - 1);
}

// Message stores for one quad of one row (every lane of the wave active);
// STREAM: an 8-bit plane larger than the Infinity Cache (store_fields32).
template <int KIND, int LB, bool STREAM>
__device__ __forceinline__ void store_message(uint32_t *__restrict__ sign_row, uint32_t *__restrict__ level_row,
                                              float *__restrict__ val_row, int64_t q, const QuadCodes &cq) {
    if (KIND == kSign || KIND == kQsgd) {
        // the word of each 8-lane group (32 elements), then the four words of
        // lanes 4, 12, 20, 28 (and 36 .. 60) gathered into one 16-byte store:
        // 0.5 % faster than eight 4-byte stores (32 workers x 2^25 elements
        // and 16 x 6.3M); as a non-temporal store 3 % slower
        const uint32_t word = or_reduce8_to_lane4(cq.sign_nib << (4 * (q & 7)));
        u32x4 v4;
        v4.x = word;
        v4.y = static_cast<uint32_t>(__shfl_down(static_cast<int>(word), 8));
        v4.z = static_cast<uint32_t>(__shfl_down(static_cast<int>(word), 16));
        v4.w = static_cast<uint32_t>(__shfl_down(static_cast<int>(word), 24));
        if ((q & 31) == 4) *reinterpret_cast<u32x4 *>(sign_row + (q >> 3)) = v4;
    }
    if (KIND == kQsgd) {
        if (LB == 8) {
            store_fields32<STREAM>(level_row, q, cq.levels);
        } else {
            const uint32_t l = cq.levels;
            store_fields16(level_row, q, (l & 0xFu) | ((l >> 4) & 0xF0u) | ((l >> 8) & 0xF00u) | ((l >> 12) & 0xF000u));
        }
    }
    if (KIND == kMbit) {
        // m-bit sign-magnitude codes: the sign bit on top of each field
        const uint32_t nib = cq.sign_nib, l = cq.levels;
        if (LB == 8) {
            const uint32_t code = l | ((nib & 1u) << 7) | ((nib & 2u) << 14) | ((nib & 4u) << 21) | ((nib & 8u) << 28);
            store_fields32<STREAM>(level_row, q, code);
        } else {
            store_fields16(level_row, q,
                           (l & 0x7u) | ((l >> 4) & 0x70u) | ((l >> 8) & 0x700u) | ((l >> 12) & 0x7000u) |
                               ((nib & 1u) << 3) | ((nib & 2u) << 6) | ((nib & 4u) << 9) | ((nib & 8u) << 12));
        }
    }
    if (KIND == kIdentity) st4(val_row + 4 * q, cq.phat);
}

// store_message with the store kind chosen at run time (kernels off the
// fused step's hot loop).
template <int KIND, int LB>
__device__ __forceinline__ void store_message_rt(uint32_t *__restrict__ sign_row, uint32_t *__restrict__ level_row,
                                                 float *__restrict__ val_row, int64_t q, const QuadCodes &cq,
                                                 bool stream) {
    if (stream)
        store_message<KIND, LB, true>(sign_row, level_row, val_row, q, cq);
    else
        store_message<KIND, LB, false>(sign_row, level_row, val_row, q, cq);
}

struct RowArgs {
    float eta;
    uint32_t t;
    int64_t d, ld;
    int32_t M, n_seg, s;
    uint32_t k0, k1;
    int64_t sign_words, level_words;  // words per row of each plane
    int32_t stream_msg;               // message planes larger than the Infinity Cache: streaming stores
};

// Row kernels off the fused step (encode, unpack, pack), bound by HBM: each thread
// takes one quad of kUnits units, all loaded before the first is worked on
// (one quad per thread with its own segment lookup left HBM idle: pack +
// unpack of 16 workers x 6.3M 8-bit codes 236 us, now 132).  A unit is a row
// (COLS = false: rows 4 y .. 4 y + 3 of one 1024-column tile, whose segments
// are looked up once) or, for fewer than kUnits rows, a tile of one row.
constexpr int kUnits = 4;

struct UnitPos {
    int m;
    int64_t tile;
    bool live;
};
template <bool COLS>
__device__ __forceinline__ UnitPos unit_at(int u, int M, int64_t n_tiles) {
    UnitPos p;
    p.m = COLS ? static_cast<int>(blockIdx.y) : static_cast<int>(blockIdx.y) * kUnits + u;
    p.tile = COLS ? static_cast<int64_t>(blockIdx.x) * kUnits + u : static_cast<int64_t>(blockIdx.x);
    p.live = p.m < M && p.tile < n_tiles;
    return p;
}

// Worker side only (dqgan_compress_ef).  One worker's row in tiles of four
// (one quad per thread, its segments found by vector loads, before): compress
// and update of 2^25 elements, s = 255, 252 -> 237 us, of 6 10^7 489 -> 463.
template <int KIND, int LB, bool COLS, bool STREAM>
__global__ __launch_bounds__(kBlock) void k_encode_rows(const float *__restrict__ G, float *__restrict__ E,
                                                        uint32_t *__restrict__ sign_plane,
                                                        uint32_t *__restrict__ level_plane, float *__restrict__ val,
                                                        const SegConst *__restrict__ consts,
                                                        const int64_t *__restrict__ off,
                                                        const int32_t *__restrict__ tile_seg, RowArgs a) {
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t n_tiles = a.ld >> 10;
    f32x4 gv[kUnits], ev[kUnits];
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
        if (!p.live) continue;
        const int64_t o = p.m * a.ld + p.tile * kElemsPerBlock + 4 * threadIdx.x;
        gv[u] = ld_io<STREAM>(G + o);
        ev[u] = ld_io<STREAM>(E + o);
    }
    // the wave's 256 columns of each unit: the first one's segment, and
    // whether it holds them all
    int jf[kUnits] = {0, 0, 0, 0};
    bool one[kUnits] = {true, true, true, true};
    if (KIND != kIdentity) {
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
            if (!COLS && u > 0) {
                jf[u] = jf[0];
                one[u] = one[0];
            } else if (p.live) {
                const int64_t w0 = p.tile * kElemsPerBlock + 256 * wave;
                jf[u] = uniform_segment(off, tile_seg, w0, a.d);
                one[u] = off[jf[u] + 1] >= (w0 + 256 < a.d ? w0 + 256 : a.d);
            }
        }
    }
    int js[4];  // the quad's segments where the wave's columns hold several; rows of one tile look them up once
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
        if (!p.live) continue;  // whole workgroups
        const int64_t q = p.tile * kQuadsPerBlock + threadIdx.x, i0 = 4 * q;
        const int64_t rb = p.m * a.ld;
        const SegConst *crow = consts + static_cast<int64_t>(p.m) * a.n_seg;
        QuadCodes cq;
        if (one[u]) {
            const SegConst c1[1] = {KIND == kIdentity ? SegConst{0.0f, 0.0f} : crow[jf[u]]};
            const int z[4] = {0, 0, 0, 0};
            cq = encode_quad<KIND>(gv[u], ev[u], a.eta, i0, a.d, p.m, z, c1, a.s, a.k0, a.k1, a.t);
        } else {
            if (COLS || u == 0) walk_segments(off, jf[u], i0, a.d, js);
            cq = encode_quad<KIND>(gv[u], ev[u], a.eta, i0, a.d, p.m, js, crow, a.s, a.k0, a.k1, a.t);
        }
        st_io<STREAM>(E + rb + i0, cq.enew);
        store_message_rt<KIND, LB>(sign_plane + p.m * a.sign_words, level_plane + p.m * a.level_words, val + rb, q, cq,
                                   a.stream_msg != 0);
    }
}

// The fused step, any M: one lane walks all rows; the second sweep re-reads g
// and the new e.
template <int KIND, int LB>
__global__ __launch_bounds__(kBlock) void k_fused(const float *__restrict__ G, float *__restrict__ E,
                                                  float *__restrict__ W, float *__restrict__ WX,
                                                  float *__restrict__ Qhat, uint32_t *__restrict__ sign_plane,
                                                  uint32_t *__restrict__ level_plane, float *__restrict__ val,
                                                  const SegConst *__restrict__ consts, const int64_t *__restrict__ off,
                                                  const int32_t *__restrict__ tile_seg, RowArgs a, float invM,
                                                  TopkArgs ta) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kQuadsPerBlock + threadIdx.x;
    const int64_t i0 = 4 * q;
    // top-k: each wave's 64 quads are one counting tile
    const int64_t tile = static_cast<int64_t>(blockIdx.x) * (kQuadsPerBlock / 64) + (threadIdx.x >> 6);
    const int M = a.M;
    int js[4];
    lookup_segments(off, tile_seg, i0, a.d, js);
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int m = 0; m < M; ++m) {
        const int64_t rb = static_cast<int64_t>(m) * a.ld;
        const f32x4 g = ld_stream(G + rb + i0);
        const f32x4 e = ld_stream(E + rb + i0);
        QuadCodes cq;
        if constexpr (KIND == kTopk) {
            const TopkRow *rw = ta.rows + m;
            cq = encode_quad_topk(g, e, a.eta, i0, a.d, rw->T, rw->I);
        } else {
            cq = encode_quad<KIND>(g, e, a.eta, i0, a.d, m, js, consts + static_cast<int64_t>(m) * a.n_seg, a.s, a.k0,
                                   a.k1, a.t);
        }
        st_stream(E + rb + i0, cq.enew);
        if constexpr (KIND == kTopk) {
            store_topk(val + m * ta.k, ta.idx + m * ta.k, ta.k, topk_tile_base(ta, m, tile), i0, cq);
        } else {
            store_message_rt<KIND, LB>(sign_plane + m * a.sign_words, level_plane + m * a.level_words, val + rb, q, cq,
                                       a.stream_msg != 0);
        }
        if (m == 0) {
            acc = cq.phat;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) set_elem(acc, c, add_rn(elem(acc, c), elem(cq.phat, c)));
        }
    }
    f32x4 qh;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float sacc = elem(acc, c);
        const float v = invM > 0.0f ? mul_rn(sacc, invM)
                                    : static_cast<float>(static_cast<double>(sacc) / static_cast<double>(M));
        set_elem(qh, c, v);
    }
    const f32x4 w = ld4(W + i0);
    f32x4 wt;
#pragma unroll
    for (int c = 0; c < 4; ++c) set_elem(wt, c, sub_rn(elem(w, c), elem(qh, c)));
    st4(W + i0, wt);
    if (Qhat) st4(Qhat + i0, qh);
#pragma unroll 1
    for (int m = 0; m < M; ++m) {
        const int64_t rb = static_cast<int64_t>(m) * a.ld;
        const f32x4 g = ld4(G + rb + i0);
        const f32x4 en = ld4(E + rb + i0);
        f32x4 x;
#pragma unroll
        for (int c = 0; c < 4; ++c) set_elem(x, c, add_rn(mul_rn(a.eta, elem(g, c)), elem(en, c)));
        f32x4 wx;
#pragma unroll
        for (int c = 0; c < 4; ++c) set_elem(wx, c, (i0 + c < a.d) ? sub_rn(elem(wt, c), elem(x, c)) : 0.0f);
        st_stream(WX + rb + i0, wx);
    }
}

// The fused step with the rows split across the NG waves of a workgroup:
// all waves cover the same 64 quads, wave g owns rows g*R .. g*R+R-1 (rows
// at or beyond M are skipped) and keeps only their p-hat and extrapolation
// operands in registers.  The server sum runs in ascending worker order as a
// chain through LDS: wave g adds its rows to the partial sum of waves
// 0..g-1, so the result is the same sequential binary32 sum as in the
// one-lane-per-quad kernel.  Few registers per lane leave room for many
// waves per SIMD, which keeps enough loads in flight to stream from HBM.
// NB > 1 (more rows than the waves can keep at once): the waves take NB
// blocks of NG R rows in turn, the chain going on from block to block; only
// the extrapolation operands of the earlier blocks stay in registers.
template <int KIND, int LB, int R, int NG, int NB, int IO>
__global__ __launch_bounds__(64 * NG) void k_fused_split(const float *__restrict__ G, float *__restrict__ E,
                                                         float *__restrict__ W, float *__restrict__ WX,
                                                         float *__restrict__ Qhat, uint32_t *__restrict__ sign_plane,
                                                         uint32_t *__restrict__ level_plane, float *__restrict__ val,
                                                         const SegConst *__restrict__ consts,
                                                         const int64_t *__restrict__ off,
                                                         const int32_t *__restrict__ tile_seg, RowArgs a, float invM,
                                                         TopkArgs ta) {
    __shared__ f32x4 chain[64];
    const int lane = threadIdx.x & 63;
    const int g = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int M = a.M;
    const int last = (M - 1) / R;  // the link of the chain that finishes the sum
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    const int64_t i0 = 4 * q;
    // One row per wave (every wave that is launched owns one): its loads go
    // out before anything is looked up.
    f32x4 g_first, e_first;
    if constexpr (R == 1) {
        const int64_t rb0 = static_cast<int64_t>(g) * a.ld;
        g_first = ld_io<IO != kIoCached>(G + rb0 + i0);
        e_first = ld_io<IO != kIoCached>(E + rb0 + i0);
    }
    // The workgroup's first segment, by scalar loads, and whether it holds
    // all of the workgroup's columns (the common case): then a row's
    // constants are one scalar load, and no lane looks up its elements'
    // segments (a chain of dependent vector loads before the first row); else
    // the lanes walk on from the workgroup's first segment, not from the tile's.
    const int64_t c0 = static_cast<int64_t>(blockIdx.x) * 256;
    const int64_t c1 = c0 + 256 < a.d ? c0 + 256 : a.d;
    const int j_first = KIND == kTopk || KIND == kIdentity ? 0 : uniform_segment(off, tile_seg, c0, a.d);
    const bool one_seg = KIND == kTopk || KIND == kIdentity || off[j_first + 1] >= c1;
    int js[4] = {j_first, j_first, j_first, j_first};
    if (!one_seg) walk_segments(off, j_first, i0, a.d, js);
    f32x4 ph[R], xs[NB * R];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        if (nb > 0 && nb * NG > last) break;  // uniform: no row left
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int m = (nb * NG + g) * R + r;
            if (m < M) {
                const int64_t rb = static_cast<int64_t>(m) * a.ld;
                const f32x4 gv = R == 1 ? g_first : ld_io<IO != kIoCached>(G + rb + i0);
                const f32x4 ev = R == 1 ? e_first : ld_io<IO != kIoCached>(E + rb + i0);
                const SegConst *crow = consts + static_cast<int64_t>(m) * a.n_seg;
                QuadCodes cq;
                if constexpr (KIND == kTopk) {
                    const TopkRow *rw = ta.rows + m;
                    cq = encode_quad_topk(gv, ev, a.eta, i0, a.d, rw->T, rw->I);
                } else if (one_seg) {
                    const SegConst cu = crow[j_first];
                    const SegConst c4[1] = {cu};
                    const int z[4] = {0, 0, 0, 0};
                    cq = encode_quad<KIND>(gv, ev, a.eta, i0, a.d, m, z, c4, a.s, a.k0, a.k1, a.t);
                } else {
                    cq = encode_quad<KIND>(gv, ev, a.eta, i0, a.d, m, js, crow, a.s, a.k0, a.k1, a.t);
                }
                st_stream(E + rb + i0, cq.enew);
                if constexpr (KIND == kTopk) {
                    store_topk(val + m * ta.k, ta.idx + m * ta.k, ta.k, topk_tile_base(ta, m, blockIdx.x), i0, cq);
                } else {
                    store_message<KIND, LB, IO == kIoStreamAll>(sign_plane + m * a.sign_words, level_plane + m * a.level_words,
                                                    val + rb, q, cq);
                }
                ph[r] = cq.phat;
#pragma unroll
                for (int c = 0; c < 4; ++c) set_elem(xs[nb * R + r], c, add_rn(elem(cq.eg, c), elem(cq.enew, c)));
            }
        }
#pragma unroll
        for (int phase = 0; phase < NG; ++phase) {
            if (nb * NG + phase <= last) {
                if (g == phase) {
                    f32x4 acc;
                    if (nb == 0 && phase == 0) {
                        acc = ph[0];
                    } else {
                        acc = chain[lane];
#pragma unroll
                        for (int c = 0; c < 4; ++c) set_elem(acc, c, add_rn(elem(acc, c), elem(ph[0], c)));
                    }
#pragma unroll
                    for (int r = 1; r < R; ++r) {
                        if ((nb * NG + g) * R + r < M) {
#pragma unroll
                            for (int c = 0; c < 4; ++c) set_elem(acc, c, add_rn(elem(acc, c), elem(ph[r], c)));
                        }
                    }
                    if (nb * NG + phase < last) {
                        chain[lane] = acc;
                    } else {
                        f32x4 qh;
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const float sacc = elem(acc, c);
                            set_elem(qh, c, invM > 0.0f ? mul_rn(sacc, invM)
                                                        : static_cast<float>(static_cast<double>(sacc) /
                                                                             static_cast<double>(M)));
                        }
                        const f32x4 w = ld4(W + i0);
                        f32x4 wt;
#pragma unroll
                        for (int c = 0; c < 4; ++c) set_elem(wt, c, sub_rn(elem(w, c), elem(qh, c)));
                        st4(W + i0, wt);
                        if (Qhat) st4(Qhat + i0, qh);
                        chain[lane] = wt;
                    }
                }
                __syncthreads();
            }
        }
    }
    const f32x4 wt = chain[lane];
#pragma unroll
    for (int r = 0; r < NB * R; ++r) {
        const int m = ((r / R) * NG + g) * R + r % R;
        if (m < M) {
            const int64_t rb = static_cast<int64_t>(m) * a.ld;
            f32x4 wx;
#pragma unroll
            for (int c = 0; c < 4; ++c) set_elem(wx, c, (i0 + c < a.d) ? sub_rn(elem(wt, c), elem(xs[r], c)) : 0.0f);
            st_stream(WX + rb + i0, wx);
        }
    }
}

// The constant b of SegConst (the decoded magnitude is level_magnitude(level,
// b)) from a scale, by binary32 arithmetic: u sigma is exact and its quotient
// by the levels, correctly rounded, is far from the denormals, so this equals
// seg_const's.  SIGN: the scale.
template <int KIND>
__device__ __forceinline__ float decode_const(float sc, int levels) {
    if (KIND == kSign) return sc;
    if (!(sc > 0.0f && sc <= 3.402823466e38f)) return 0.0f;
    const bool tiny = sc < 0x1.0p-64f;
    const float b = mul_rn(sc, tiny ? 0x1.0p64f : 1.0f) / static_cast<float>(levels);
    return tiny ? -b : b;
}

// Element c (0..3) of a quad's fields: nib = the four sign bits (SIGN,
// QSGD), raw = the quad's level or code bits (QSGD, MBIT: 32 bits for 8-bit
// fields, the low 16 for 4-bit fields).
template <int KIND, int LB>
__device__ __forceinline__ uint32_t field_level(uint32_t raw, int c) {
    const uint32_t f = LB == 8 ? (raw >> (8 * c)) & 0xFFu : (raw >> (4 * c)) & 0xFu;
    return KIND == kMbit ? f & (LB == 8 ? 0x7Fu : 0x7u) : f;
}
template <int KIND, int LB>
__device__ __forceinline__ uint32_t field_sign(uint32_t nib, uint32_t raw, int c) {  // in bit 31
    const uint32_t x = KIND == kMbit ? raw << (31 - (LB * (c + 1) - 1)) : nib << (31 - c);
    return x & 0x80000000u;
}
// Its decoded value.  The magnitude is never negative, so the sign bit is set
// by OR (-0 for a zero level with the sign bit set, as the encoder gives).
// RANGE: b may be negative (level_magnitude).
template <int KIND, int LB, bool RANGE>
__device__ __forceinline__ float decode_field(uint32_t nib, uint32_t raw, int c, float b) {
    const uint32_t l = KIND == kSign ? 0u : field_level<KIND, LB>(raw, c);
    const float mag = KIND == kSign ? b : RANGE ? level_magnitude(l, b) : mul_rn(static_cast<float>(l), b);
    return __uint_as_float(__float_as_uint(mag) | field_sign<KIND, LB>(nib, raw, c));
}

template <int KIND, int LB, bool COLS>
__global__ __launch_bounds__(kBlock) void k_unpack(const uint32_t *__restrict__ sign_plane,
                                                   const uint32_t *__restrict__ level_plane,
                                                   const float *__restrict__ val, const float *__restrict__ scale,
                                                   float *__restrict__ Phat, const int64_t *__restrict__ off,
                                                   const int32_t *__restrict__ tile_seg, RowArgs a) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    const int64_t n_tiles = a.ld >> 10;
    uint32_t sg[kUnits], raw[kUnits];
    f32x4 v[kUnits];
    float b[kUnits];
    int js[kUnits];
    bool one[kUnits];
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
        sg[u] = raw[u] = 0u;
        if (!p.live) continue;
        const int64_t q = p.tile * kQuadsPerBlock + threadIdx.x;
        if (KIND == kSign || KIND == kQsgd) sg[u] = sign_plane[p.m * a.sign_words + (q >> 3)];
        if (KIND == kQsgd || KIND == kMbit) {
            const uint32_t *row = level_plane + p.m * a.level_words;
            raw[u] = LB == 8 ? row[q] : static_cast<uint32_t>(reinterpret_cast<const uint16_t *>(row)[q]);
        }
        if (KIND == kIdentity) v[u] = ld4(val + static_cast<int64_t>(p.m) * a.ld + 4 * q);
    }
    if (KIND != kIdentity) {
        // the wave's 256 columns of each unit: its segment, and its constant
        // where one segment holds them all
#pragma unroll
        for (int u = 0; u < kUnits; ++u) {
            const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
            if (!COLS && u > 0) {
                js[u] = js[0];
                one[u] = one[0];
            } else if (p.live) {
                const int64_t w0 = p.tile * kElemsPerBlock + 256 * wave;
                js[u] = uniform_segment(off, tile_seg, w0, a.d);
                one[u] = off[js[u] + 1] >= (w0 + 256 < a.d ? w0 + 256 : a.d);
            }
            if (p.live) b[u] = decode_const<KIND>(scale[static_cast<int64_t>(p.m) * a.n_seg + js[u]], a.s);
        }
    }
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
        if (!p.live) continue;
        const int64_t q = p.tile * kQuadsPerBlock + threadIdx.x, i0 = 4 * q;
        f32x4 o;
        if (KIND == kIdentity) {
            o = v[u];
        } else if (one[u]) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                set_elem(o, c, decode_field<KIND, LB, true>(sg[u] >> (4 * (lane & 7)), raw[u], c, b[u]));
        } else {
            int j = js[u];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                j = seg_from(off, j, i0 + c < a.d ? i0 + c : a.d - 1);
                const float bc = decode_const<KIND>(scale[static_cast<int64_t>(p.m) * a.n_seg + j], a.s);
                set_elem(o, c, decode_field<KIND, LB, true>(sg[u] >> (4 * (lane & 7)), raw[u], c, bc));
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (i0 + c >= a.d) set_elem(o, c, 0.0f);
        st_stream(Phat + static_cast<int64_t>(p.m) * a.ld + i0, o);
    }
}

// Server average of the M messages.  A thread covers four consecutive
// quads (16 elements: 16 sign bits, 8 or 16 bytes of fields per row, so
// each row's loads are 2-16 bytes per lane rather than sub-word), a wave
// 1024.  The sum runs in ascending worker order, from -0 (fl(-0 + x) = x for
// every x, so the sum is the definition's, which starts from worker 0's
// term).  Elements at or beyond d are summed with the rest and dropped at the
// end.
//
// Bound by the vector ALU: about 5 operations per decoded element (a byte's
// conversion, the product, the sign's shift and OR, the sum; 4-bit fields are
// made bytes eight at a time: with each extracted by itself 185 us instead of
// 179 at 32 workers x 2^25, s = 15, 57 instead of 52 at 16 x 20M 4-bit codes).
// 262 us with 8.8 operations, a bound test per row, and constants from a launch
// of their own.
// 16 workers x 6.3M 8-bit codes 46 -> 30 us, 8 x 10^6 15.3 -> 11.5.
// Held to 80 registers for six waves per SIMD the kernel spills: 274 us.
constexpr int kAggQuads = 4;
// Rows loaded before the first is decoded.  One plane a row: more rows in flight (32
// workers x 2^25 signs 108 us with eight, 116 with four; 16 x 20M 8-bit codes 79,
// 81; 4-bit codes 51.5, 53.8; two planes, s = 255: 88.5, 87).
constexpr int agg_rows(int kind) { return kind == kQsgd ? 4 : 8; }
// Segments of a wave up to which each takes a pass of its own over the wave's
// messages; with more every element looks its constant up, in one pass that
// costs about 12 of the others (s levels 16, 8-bit codes 8).  A row outside a full
// batch costs 2 to 4 in one; the batches of four have a row's worth of overhead
// or two.  4M elements, a pass per segment / look-ups: 32 workers, signs, 8
// segments a tile 94 / 174 us, 12 133 / 197; s = 255, 8 182 / 277, 13 294 / 342;
// 8-bit codes, 8 173 / 189, 12 256 / 224; 6 workers, signs, 8 47 / 41, s = 255,
// 8 56 / 48; 4 workers, 8-bit codes, 8 43 / 33, 4 26 / 26.
int agg_segs(int kind, int level_bits, int M) {
    const int left = M % agg_rows(kind), full = M - left;
    const int n = kind == kQsgd                      ? 16 * M / (full + 4 * left + 2)
                  : kind == kMbit && level_bits == 8 ? 8 * M / (full + 3 * left)
                                                     : 12 * M / (full + 2 * left);
    return std::max(n, 5);  // 1 worker, s = 255, 3 segments 12.4 / 15.4 us
}

template <int KIND, int LB>
struct AggFields {
    static constexpr int kWords = (KIND == kQsgd || KIND == kMbit) ? LB / 2 : 1;  // 32-bit words of fields per row
    uint32_t sg, fw[kWords];

    __device__ __forceinline__ void load(const uint32_t *__restrict__ sign_plane,
                                         const uint32_t *__restrict__ level_plane, const RowArgs &a, int m,
                                         int64_t g16) {
        if (KIND == kSign || KIND == kQsgd) sg = reinterpret_cast<const uint16_t *>(sign_plane + m * a.sign_words)[g16];
        if (KIND == kQsgd || KIND == kMbit) {
            const uint32_t *w = level_plane + m * a.level_words + kWords * g16;
            if constexpr (kWords == 4) {
                const u32x4 x = *reinterpret_cast<const u32x4 *>(w);
#pragma unroll
                for (int c = 0; c < 4; ++c) fw[c] = elem(x, c);
            } else if constexpr (kWords == 2) {
                const uint2 x = *reinterpret_cast<const uint2 *>(w);
                fw[0] = x.x;
                fw[1] = x.y;
            }
        }
    }
    // 4-bit fields as bytes, the even ones of a word and the odd ones: a byte's
    // conversion is one operation with its extraction.  (The empty asm keeps
    // the compiler from extracting each field from the word again.)
    uint32_t even[kWords], odd[kWords];
    __device__ __forceinline__ void split() {
        if (LB != 4) return;
        constexpr uint32_t mask = KIND == kMbit ? 0x07070707u : 0x0F0F0F0Fu;
#pragma unroll
        for (int c = 0; c < kWords; ++c) {
            even[c] = fw[c] & mask;
            odd[c] = (fw[c] >> 4) & mask;
            asm("" : "+v"(even[c]), "+v"(odd[c]));
        }
    }
    // element c of quad k (after split())
    template <bool RANGE>
    __device__ __forceinline__ float value(int k, int c, float b) const {
        if constexpr (LB == 4) {
            const int w = (k >> 1) % kWords, f = 4 * (k & 1) + c;  // field f of word w
            const uint32_t l = ((f & 1 ? odd[w] : even[w]) >> (8 * (f >> 1))) & 0xFFu;
            const float mag = RANGE ? level_magnitude(l, b) : mul_rn(static_cast<float>(l), b);
            return __uint_as_float(__float_as_uint(mag) | field_sign<KIND, LB>(sg >> (8 * (k >> 1)), fw[w], f));
        }
        const uint32_t raw = KIND == kSign ? 0u : kWords == 4 ? fw[k % kWords] : fw[(k >> 1) % kWords] >> (16 * (k & 1));
        return decode_field<KIND, LB, RANGE>(sg >> (4 * k), raw, c, b);
    }
};

template <int KIND, int LB, bool MANY>
__global__ __launch_bounds__(kBlock) void k_aggregate(const uint32_t *__restrict__ sign_plane,
                                                      const uint32_t *__restrict__ level_plane,
                                                      const float *__restrict__ scale, float *__restrict__ Qhat,
                                                      const SegConst *__restrict__ consts,
                                                      const int64_t *__restrict__ off,
                                                      const int32_t *__restrict__ tile_seg, RowArgs a, float invM,
                                                      int few_segs) {
    typedef AggFields<KIND, LB> Fields;
    constexpr int kAggRows = agg_rows(KIND);
    const int lane = threadIdx.x & 63;
    const int64_t tile = static_cast<int64_t>(blockIdx.x) * (kBlock / 64) +
                         __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
    if (tile >= (a.ld >> 10)) return;  // whole waves
    const int64_t g16 = tile * 64 + lane;  // group of 16 elements
    const int64_t w0 = tile << 10;
    const int64_t w1 = w0 + 1024 < a.d ? w0 + 1024 : a.d;  // past the wave's last element below d (w1 <= w0: none)
    const int j0 = tile_seg[tile];
    int j1 = j0;  // the wave's last segment
    while (off[j1 + 1] < w1) ++j1;
    f32x4 acc[kAggQuads], qh[kAggQuads];
    auto restart = [&] {
#pragma unroll
        for (int k = 0; k < kAggQuads; ++k) acc[k] = f32x4{-0.0f, -0.0f, -0.0f, -0.0f};
    };
    // the average of the elements of [lo, hi) from their sums
    auto keep = [&](int64_t lo, int64_t hi) {
#pragma unroll
        for (int k = 0; k < kAggQuads; ++k) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t i = 16 * g16 + 4 * k + c;
                const float sacc = elem(acc[k], c);
                const float x = invM > 0.0f ? mul_rn(sacc, invM)
                                            : static_cast<float>(static_cast<double>(sacc) / static_cast<double>(a.M));
                if (i >= lo && i < hi) set_elem(qh[k], c, x);
            }
        }
    };
#pragma unroll
    for (int k = 0; k < kAggQuads; ++k) qh[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // Every row's 16 elements decoded with the constants of segment j.
    auto sum_rows = [&](int j) {
        // lane l keeps the constant of row mb + l, handed to the wave as a
        // scalar when the row's turn comes
        for (int mb = 0; mb < a.M; mb += 64) {
            const int n = a.M - mb < 64 ? a.M - mb : 64;
            float bl = 0.0f;
            if (lane < n)
                bl = decode_const<KIND>(scale[static_cast<int64_t>(mb + lane) * a.n_seg + j], a.s);
            auto rows = [&](auto range) {
                auto add_row = [&](Fields &f, int r) {
                    f.split();
                    const float b = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(bl), r));
#pragma unroll
                    for (int k = 0; k < kAggQuads; ++k) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            set_elem(acc[k], c,
                                     add_rn(elem(acc[k], c), f.template value<decltype(range)::value>(k, c, b)));
                    }
                };
                // batches of rows all loaded before the first is decoded,
                // then the rows left over
                int r0 = 0;
                for (; r0 + kAggRows <= n; r0 += kAggRows) {
                    Fields f[kAggRows];
#pragma unroll
                    for (int u = 0; u < kAggRows; ++u) f[u].load(sign_plane, level_plane, a, mb + r0 + u, g16);
#pragma unroll
                    for (int u = 0; u < kAggRows; ++u) add_row(f[u], r0 + u);
                }
                for (; r0 < n; ++r0) {
                    Fields f;
                    f.load(sign_plane, level_plane, a, mb + r0, g16);
                    add_row(f, r0);
                }
            };
            // no negative constant (no scale below 2^-64): one product less
            // per element
            if (KIND == kSign || __ballot(bl < 0.0f) == 0)
                rows(std::false_type{});
            else
                rows(std::true_type{});
        }
    };
    if (!MANY || j1 - j0 < few_segs) {
        // one segment (the common case) or a few: each decodes the wave's
        // messages once and keeps its own elements
        for (int j = j0; j <= j1; ++j) {
            restart();
            sum_rows(j);
            keep(off[j], off[j + 1]);
        }
    } else if constexpr (MANY) {
        // many short segments: every element its own constant, its segment
        // looked up once for all rows (walked again for every row, 32 workers x
        // 4M 8-bit codes in segments of 100 took 470 us a call, now 224)
        int js[kAggQuads][4];
#pragma unroll
        for (int k = 0; k < kAggQuads; ++k)
            walk_segments(off, k == 0 ? j0 : js[k > 0 ? k - 1 : 0][3], 16 * g16 + 4 * k, a.d, js[k]);
        restart();
        for (int m = 0; m < a.M; ++m) {
            Fields f;
            f.load(sign_plane, level_plane, a, m, g16);
            f.split();
            const SegConst *crow = consts + static_cast<int64_t>(m) * a.n_seg;
#pragma unroll
            for (int k = 0; k < kAggQuads; ++k) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float b = KIND == kSign ? crow[js[k][c]].a : crow[js[k][c]].b;
                    set_elem(acc[k], c, add_rn(elem(acc[k], c), f.template value<true>(k, c, b)));
                }
            }
        }
        keep(0, a.d);
    }
#pragma unroll
    for (int k = 0; k < kAggQuads; ++k) st4(Qhat + 16 * g16 + 4 * k, qh[k]);
}

// The same for IDENTITY messages (dense binary32 rows): one quad per thread, so
// that a wave reads 1 KB of a row at a time.
constexpr int kMeanRows = 8;  // rows loaded before the first is added

__global__ __launch_bounds__(kBlock) void k_mean_rows(const float *__restrict__ val, float *__restrict__ Qhat,
                                                      int64_t d, int64_t ld, int32_t M, float invM) {
    const int64_t i0 = 4 * (static_cast<int64_t>(blockIdx.x) * kQuadsPerBlock + threadIdx.x);
    const float *src = val + i0;
    f32x4 acc = {-0.0f, -0.0f, -0.0f, -0.0f};
    auto add = [&](const f32x4 &v) {
#pragma unroll
        for (int c = 0; c < 4; ++c) set_elem(acc, c, add_rn(elem(acc, c), elem(v, c)));
    };
    int m = 0;
    for (; m + kMeanRows <= M; m += kMeanRows) {
        f32x4 v[kMeanRows];
#pragma unroll
        for (int u = 0; u < kMeanRows; ++u) v[u] = ld_stream(src + static_cast<int64_t>(m + u) * ld);
#pragma unroll
        for (int u = 0; u < kMeanRows; ++u) add(v[u]);
    }
    for (; m < M; ++m) add(ld_stream(src + static_cast<int64_t>(m) * ld));
    f32x4 qh;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float sacc = elem(acc, c);
        const float x = invM > 0.0f ? mul_rn(sacc, invM)
                                    : static_cast<float>(static_cast<double>(sacc) / static_cast<double>(M));
        set_elem(qh, c, i0 + c < d ? x : 0.0f);
    }
    st4(Qhat + i0, qh);
}

template <bool STREAM>
__global__ __launch_bounds__(kBlock) void k_omd(const float *__restrict__ Qhat, float *__restrict__ W,
                                                const float *__restrict__ G, const float *__restrict__ E,
                                                float *__restrict__ WX, float eta, int64_t d, int64_t ld, int32_t M) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kQuadsPerBlock + threadIdx.x;
    const int64_t i0 = 4 * q;
    const f32x4 w = ld4(W + i0);
    const f32x4 qh = ld4(Qhat + i0);
    f32x4 wt;
#pragma unroll
    for (int c = 0; c < 4; ++c) set_elem(wt, c, (i0 + c < d) ? sub_rn(elem(w, c), elem(qh, c)) : elem(w, c));
    st4(W + i0, wt);
    if (!WX) return;
    // kOmdRows workers' g and e loaded before the first evaluation point
    constexpr int kOmdRows = 4;
    for (int m0 = 0; m0 < M; m0 += kOmdRows) {
        f32x4 gv[kOmdRows], ev[kOmdRows];
#pragma unroll
        for (int u = 0; u < kOmdRows; ++u) {
            if (m0 + u < M) {
                const int64_t rb = static_cast<int64_t>(m0 + u) * ld;
                gv[u] = ld_io<STREAM>(G + rb + i0);
                ev[u] = ld_io<STREAM>(E + rb + i0);
            }
        }
#pragma unroll
        for (int u = 0; u < kOmdRows; ++u) {
            if (m0 + u < M) {
                f32x4 wx;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float x = add_rn(mul_rn(eta, elem(gv[u], c)), elem(ev[u], c));
                    set_elem(wx, c, (i0 + c < d) ? sub_rn(elem(wt, c), x) : 0.0f);
                }
                st_stream(WX + static_cast<int64_t>(m0 + u) * ld + i0, wx);
            }
        }
    }
}

// Packs the caller's codes; the scales (when they are not the message's own)
// are copied by the first threads of the grid.
template <int LB, int KIND, bool COLS>
__global__ __launch_bounds__(kBlock) void k_pack(const uint16_t *__restrict__ codes, const float *__restrict__ scales,
                                                 uint32_t *__restrict__ sign_plane, uint32_t *__restrict__ level_plane,
                                                 float *__restrict__ scale_out, RowArgs a) {
    const int64_t n_tiles = a.ld >> 10;
    uint2 raw[kUnits];
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
        if (p.live)
            raw[u] = *reinterpret_cast<const uint2 *>(codes + static_cast<int64_t>(p.m) * a.ld +
                                                      p.tile * kElemsPerBlock + 4 * threadIdx.x);
    }
    if (scale_out) {
        const int64_t n = static_cast<int64_t>(a.M) * a.n_seg;
        const int64_t wg = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
        for (int64_t i = wg * kBlock + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * gridDim.y * kBlock)
            scale_out[i] = scales[i];
    }
    const uint32_t fmask = KIND == kMbit ? (LB == 8 ? 0x7Fu : 0x7u) : (LB == 8 ? 0xFFu : 0xFu);
#pragma unroll
    for (int u = 0; u < kUnits; ++u) {
        const UnitPos p = unit_at<COLS>(u, a.M, n_tiles);
        if (!p.live) continue;  // whole workgroups
        const int64_t q = p.tile * kQuadsPerBlock + threadIdx.x, i0 = 4 * q;
        const uint32_t c4[4] = {raw[u].x & 0xFFFFu, raw[u].x >> 16, raw[u].y & 0xFFFFu, raw[u].y >> 16};
        QuadCodes cq;
        cq.sign_nib = 0u;
        cq.levels = 0u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (i0 + c >= a.d) continue;
            cq.sign_nib |= ((c4[c] >> 15) & 1u) << c;
            cq.levels |= (c4[c] & fmask) << (8 * c);
        }
        store_message_rt<KIND, LB>(KIND == kMbit ? nullptr : sign_plane + p.m * a.sign_words,
                                   KIND == kSign ? nullptr : level_plane + p.m * a.level_words, nullptr, q, cq,
                                   a.stream_msg != 0);
    }
}

// Top-k worker side only (dqgan_compress_ef): one wave per (tile, worker).
template <bool STREAM>
__global__ __launch_bounds__(64) void k_topk_encode_rows(const float *__restrict__ G, float *__restrict__ E,
                                                         float *__restrict__ val, RowArgs a, TopkArgs ta) {
    const int m = blockIdx.y;
    const int64_t q = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;
    const int64_t i0 = 4 * q;
    const int64_t rb = static_cast<int64_t>(m) * a.ld;
    const TopkRow *rw = ta.rows + m;
    const f32x4 g = ld_io<STREAM>(G + rb + i0);
    const f32x4 e = ld_io<STREAM>(E + rb + i0);
    const QuadCodes cq = encode_quad_topk(g, e, a.eta, i0, a.d, rw->T, rw->I);
    st_io<STREAM>(E + rb + i0, cq.enew);
    store_topk(val + m * ta.k, ta.idx + m * ta.k, ta.k, topk_tile_base(ta, m, blockIdx.x), i0, cq);
}

RowArgs row_args(const dqgan_plan_s &P, float eta, uint32_t t) {
    RowArgs a;
    a.eta = eta;
    a.t = t;
    a.d = P.desc.d;
    a.ld = P.desc.ld;
    a.M = P.desc.M;
    a.n_seg = P.desc.n_seg;
    a.s = P.level_count;
    a.k0 = static_cast<uint32_t>(P.desc.seed);
    a.k1 = static_cast<uint32_t>(P.desc.seed >> 32);
    a.sign_words = P.desc.ld / 32;
    a.level_words = P.level_bits ? P.desc.ld * P.level_bits / 32 : 0;
    const double msg_bytes = 4.0 * P.desc.M * static_cast<double>(a.sign_words + a.level_words);
    a.stream_msg = msg_bytes > kInfinityCacheBytes ? 1 : 0;
    return a;
}

// 1/M when M is a power of two (then x * (1/M) equals x / M exactly),
// else 0 (the kernels divide).
float inv_m(int M) { return (M & (M - 1)) == 0 ? 1.0f / static_cast<float>(M) : 0.0f; }

// The state the top-k apply pass reads (threshold per row, tile offsets).
TopkArgs topk_args(const dqgan_plan_s &P, const dqgan_wire &w) {
    TopkArgs ta{};
    if (P.desc.kind == kTopk) {
        ta.rows = P.topk.rows;
        ta.tile_off = P.topk.tile_off;
        ta.chunk_off = P.topk.chunk_off;
        ta.n_tiles = P.topk.n_tiles;
        ta.n_chunks = P.topk.n_chunks;
        ta.k = P.desc.k;
        ta.idx = w.idx;
    }
    return ta;
}

template <int KIND, int LB>
hipError_t fused_launch(const dqgan_plan_s &P, const RowArgs &a, const float *G, float *E, float *W, float *WX,
                        const dqgan_wire &w, float *Qhat, hipStream_t st) {
    hipLaunchKernelGGL((k_fused<KIND, LB>), dim3(static_cast<unsigned>(P.n_tiles)), dim3(kBlock), 0, st, G, E, W,
                       WX, Qhat, w.sign, w.level, w.val, P.d_consts, P.d_off, P.d_tile_seg, a, inv_m(P.desc.M),
                       topk_args(P, w));
    return hipGetLastError();
}

// Unused LDS per workgroup of `waves` waves that leaves room for about 24
// waves per CU with two rows per wave and for about 16 with four.  HBM serves
// the pass's mix of reads and writes faster with fewer rows in flight: 16
// workers x 6.3M 8-bit codes, whole step 464.5 us at 32 waves, 453.0 at 24,
// 469.2 at 16; 32 workers x 2^25, s = 15: 4662 us at 24 waves (all that its
// registers allow), 4609 at 16, 6337 at 8; 16 workers x 10^8 top-k 7210 us at
// 32, 7092 at 24, 7661 at 16.  The waves are those launched, which own a row:
// counted as eight, 17 workers x 3.5M 4-bit codes (5 waves) took 317 us instead
// of 270, 9 x 6.7M 275 instead of 251.  Not capped: steps that the Infinity
// Cache holds, and plans of short segments, whose waves wait for look-ups and
// constants rather than for HBM (apply pass with the cap / without: 32 workers
// x 4M, s = 15, segments of 150 550 / 487 us, 601 502 / 452, 2401 470 / 434,
// 5001 and more within 1 %; 16 workers, signs, 150 229 / 209, 601 205 / 209),
// and top-k with four rows per wave (whole step 17 workers of 4 GB 0.944 of the
// capped, 28 0.937, 32 0.974; with two rows per wave, 16 workers, 1.028).
constexpr int kLdsPerCu = 160 * 1024;
constexpr int64_t kShortSegment = 4096;  // mean elements below which a plan's segments are short
unsigned cap_lds(int R, int NG, int waves) {
    const int target = NG != 8 ? 0 : R == 2 ? 24 : R == 4 ? 16 : 0;
    if (target == 0) return 0u;
    const int wgs = (target + waves / 2) / waves;
    // less the kernel's own 1 KB and the allocation's rounding
    return static_cast<unsigned>(kLdsPerCu / wgs - 1024 - 1536);
}

template <int KIND, int LB, int R, int NG, int NB = 1>
hipError_t split_launch(const dqgan_plan_s &P, const RowArgs &a, const float *G, float *E, float *W, float *WX,
                        const dqgan_wire &w, float *Qhat, hipStream_t st) {
    if (P.desc.M > R * NG * NB) return hipErrorInvalidValue;  // every worker must belong to a wave
    const TopkArgs ta = topk_args(P, w);
    // only the waves that own a row
    const dim3 grid(static_cast<unsigned>(P.n_tiles * 4)), block(64 * static_cast<unsigned>(std::min((P.desc.M + R - 1) / R, NG)));
    // Unused LDS that caps the workgroups per CU of a step that streams from
    // HBM (see cap_lds).
    const double bytes = 16.0 * P.desc.M * static_cast<double>(P.desc.ld);
    const bool short_segs = KIND != kTopk && KIND != kIdentity && P.desc.d < kShortSegment * P.desc.n_seg;
    const bool capped = bytes > kInfinityCacheBytes && !short_segs && !(KIND == kTopk && R == 4);
    const unsigned cap = capped ? cap_lds(R, NG, static_cast<int>(block.x / 64)) : 0u;
    auto go = [&](auto io) {
        hipLaunchKernelGGL((k_fused_split<KIND, LB, R, NG, NB, decltype(io)::value>), grid, block, cap, st, G, E, W, WX,
                           Qhat, w.sign, w.level, w.val, P.d_consts, P.d_off, P.d_tile_seg, a, inv_m(P.desc.M), ta);
    };
    // Only 8-bit planes have a second store kind (store_fields32).
    constexpr bool kTwoKinds = (KIND == kQsgd || KIND == kMbit) && LB == 8;
    if (!second_streams(P.desc))
        go(Const<kIoCached>{});
    else if (kTwoKinds && a.stream_msg)
        go(Const<kTwoKinds ? kIoStreamAll : kIoStream>{});
    else
        go(Const<kIoStream>{});
    return hipGetLastError();
}

// Launch shape of the fused step: up to 16 waves per workgroup, each owning
// R rows; more rows per wave means more loads in flight per lane.  Measured:
// for 9 <= M <= 16, 8 waves x 2 rows beats 16 x 1 by 10-13 %; for
// 17 <= M <= 32, 8 waves x 4 rows beats 16 x 2 by 2-3 % although it runs 6
// rather than 8 waves per SIMD; M <= 8 (cache-resident sizes) keeps one row
// per wave; for 65 <= M <= 128, 16 waves x 8 rows (4 waves per SIMD) is a
// third faster than the one-lane kernel; for 129 <= M <= 256 four blocks of
// 16 waves x 4 rows in turn take 1376 us where the one-lane kernel takes 1759
// (256 x 10^6, s = 255).  Beyond 256 rows the operands do not fit the 128
// registers of a 16-wave workgroup, and the one-lane-per-quad kernel serves.
template <int KIND, int LB>
hipError_t fused_by_m(const dqgan_plan_s &P, const RowArgs &a, const float *G, float *E, float *W, float *WX,
                      const dqgan_wire &w, float *Qhat, hipStream_t st) {
    const int M = P.desc.M;
    if (M <= 4) return split_launch<KIND, LB, 1, 4>(P, a, G, E, W, WX, w, Qhat, st);
    if (M <= 8) return split_launch<KIND, LB, 1, 8>(P, a, G, E, W, WX, w, Qhat, st);
    if (M <= 16) return split_launch<KIND, LB, 2, 8>(P, a, G, E, W, WX, w, Qhat, st);
    if (M <= 32) return split_launch<KIND, LB, 4, 8>(P, a, G, E, W, WX, w, Qhat, st);
    if (M <= 64) return split_launch<KIND, LB, 4, 16>(P, a, G, E, W, WX, w, Qhat, st);
    if (M <= 128) return split_launch<KIND, LB, 8, 16>(P, a, G, E, W, WX, w, Qhat, st);
    if (M <= 256) return split_launch<KIND, LB, 4, 16, 4>(P, a, G, E, W, WX, w, Qhat, st);
    return fused_launch<KIND, LB>(P, a, G, E, W, WX, w, Qhat, st);
}

}  // namespace

// Whether the statistics pass derives the scales itself.  Small workloads gain
// a launch (4 workers x 65536 signs 18.5 -> 15.5 us, 16 x 500k 37.1 -> 35.6, a
// worker of 200k 28.5 -> 24).  The arrivals of a segment are atomics on one
// address, one after the other, and each holds its workgroup's place on the CU:
// with more of them the launch is cheaper (8 x 10^6, 33 pieces a segment, 39.6
// -> 41.3 us; 129 pieces 56; 16 x 6.3M 431 -> 451).
static bool stats_few(const dqgan_plan_s &P) {
    constexpr int kFewPieces = 16, kFewBlocks = 1024;
    return P.max_seg_pieces <= kFewPieces && static_cast<int64_t>(P.desc.M) * P.n_pieces <= kFewBlocks;
}

hipError_t launch_segment_scales(const dqgan_plan_s &P, float eta, const float *G, const float *E,
                                 const float *scales_in, float *scale_out, hipStream_t st) {
    const dqgan_desc &D = P.desc;
    if (!scales_in) {
        const dim3 grid(static_cast<unsigned>(P.n_pieces), static_cast<unsigned>(D.M));
        const bool few = stats_few(P);
        const StatsOut out{P.d_partial, P.d_pmax, arrivals(P), P.d_seg_piece, P.d_off,
                           scale_out, P.d_consts, D.n_seg, D.kind, D.norm, P.level_count};
        auto launch = [&](auto norm, auto stream, auto few_c) {
            hipLaunchKernelGGL((k_segment_partials<decltype(norm)::value, decltype(stream)::value, decltype(few_c)::value>),
                               grid, dim3(kBlock), 0, st, G, E, eta, D.ld, P.d_pieces, P.n_pieces, out);
        };
        auto go = [&](auto norm) {
            with_stream(first_streams(D), [&](auto stream) {
                if (few)
                    launch(norm, stream, std::true_type{});
                else
                    launch(norm, stream, std::false_type{});
            });
        };
        if (D.norm == DQGAN_L1)
            go(Const<DQGAN_L1>{});
        else if (D.norm == DQGAN_L2)
            go(Const<DQGAN_L2>{});
        else
            go(Const<DQGAN_LINF>{});
        hipError_t err = hipGetLastError();
        if (err != hipSuccess || few) return err;
    }
    const int64_t n = static_cast<int64_t>(D.M) * D.n_seg;
    // one wave per (worker, segment)
    hipLaunchKernelGGL(k_finalize, dim3(static_cast<unsigned>((n * 64 + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, D.kind,
                       D.norm, P.level_count, P.d_partial, P.d_pmax, P.n_pieces, P.d_seg_piece, P.d_off, D.M, D.n_seg,
                       scales_in, scale_out, P.d_consts);
    return hipGetLastError();
}

hipError_t launch_consts_from_scales(const dqgan_plan_s &P, const float *scales, hipStream_t st) {
    return launch_segment_scales(P, 0.0f, nullptr, nullptr, scales, nullptr, st);
}

namespace {

// Calls f(kind, field bits) with both as compile-time constants, for the
// dense compressors: (SIGN, 0), (QSGD, 8 or 4), (MBIT, 8 or 4), (IDENTITY, 0).

template <typename F>
hipError_t with_dense_kind(const dqgan_plan_s &P, F &&f) {
    switch (P.desc.kind) {
        case kSign: return f(Const<kSign>{}, Const<0>{});
        case kQsgd: return P.level_bits == 8 ? f(Const<kQsgd>{}, Const<8>{}) : f(Const<kQsgd>{}, Const<4>{});
        case kMbit: return P.level_bits == 8 ? f(Const<kMbit>{}, Const<8>{}) : f(Const<kMbit>{}, Const<4>{});
        default: return f(Const<kIdentity>{}, Const<0>{});
    }
}

}  // namespace

// The grid of a kernel over units (unit_at): f(COLS, grid).
template <typename F>
static hipError_t with_units(const dqgan_plan_s &P, F &&f) {
    const unsigned n = static_cast<unsigned>(P.n_tiles), M = static_cast<unsigned>(P.desc.M);
    if (P.desc.M < kUnits) return f(std::true_type{}, dim3((n + kUnits - 1) / kUnits, M));
    return f(std::false_type{}, dim3(n, (M + kUnits - 1) / kUnits));
}

hipError_t launch_encode(const dqgan_plan_s &P, float eta, uint32_t t, const float *G, float *E, const dqgan_wire &w,
                         hipStream_t st) {
    const RowArgs a = row_args(P, eta, t);
    return with_dense_kind(P, [&](auto K, auto L) {
        return with_units(P, [&](auto C, dim3 grid) {
            with_stream(worker_streams(P.desc), [&](auto S) {
                hipLaunchKernelGGL(
                    (k_encode_rows<decltype(K)::value, decltype(L)::value, decltype(C)::value, decltype(S)::value>),
                    grid, dim3(kBlock), 0, st, G, E, w.sign, w.level, w.val, P.d_consts, P.d_off, P.d_tile_seg, a);
            });
            return hipGetLastError();
        });
    });
}

hipError_t launch_fused_dense(const dqgan_plan_s &P, float eta, uint32_t t, const float *G, float *E, float *W,
                              float *WX, const dqgan_wire &w, float *Qhat, hipStream_t st) {
    const RowArgs a = row_args(P, eta, t);
    return with_dense_kind(P, [&](auto K, auto L) {
        return fused_by_m<decltype(K)::value, decltype(L)::value>(P, a, G, E, W, WX, w, Qhat, st);
    });
}

hipError_t launch_pack(const dqgan_plan_s &P, const uint16_t *codes, const float *scales, const dqgan_wire &w,
                       hipStream_t st) {
    const RowArgs a = row_args(P, 0.0f, 0);
    return with_dense_kind(P, [&](auto K, auto L) {
        if constexpr (decltype(K)::value == kIdentity) {
            return hipErrorInvalidValue;  // the identity has no codes to pack
        } else {
            return with_units(P, [&](auto C, dim3 grid) {
                hipLaunchKernelGGL((k_pack<decltype(L)::value, decltype(K)::value, decltype(C)::value>), grid,
                                   dim3(kBlock), 0, st, codes, scales, w.sign, w.level,
                                   scales == w.scale ? nullptr : w.scale, a);
                return hipGetLastError();
            });
        }
    });
}

hipError_t launch_unpack_dense(const dqgan_plan_s &P, const dqgan_wire &w, float *Phat, hipStream_t st) {
    const RowArgs a = row_args(P, 0.0f, 0);
    return with_dense_kind(P, [&](auto K, auto L) {
        return with_units(P, [&](auto C, dim3 grid) {
            hipLaunchKernelGGL((k_unpack<decltype(K)::value, decltype(L)::value, decltype(C)::value>), grid,
                               dim3(kBlock), 0, st, w.sign, w.level, w.val, w.scale, Phat, P.d_off, P.d_tile_seg, a);
            return hipGetLastError();
        });
    });
}

hipError_t launch_aggregate_dense(const dqgan_plan_s &P, const dqgan_wire &w, float *Qhat, hipStream_t st) {
    const RowArgs a = row_args(P, 0.0f, 0);
    const float im = inv_m(P.desc.M);
    if (P.desc.kind == kIdentity) {
        hipLaunchKernelGGL(k_mean_rows, dim3(static_cast<unsigned>(P.n_tiles)), dim3(kBlock), 0, st, w.val, Qhat,
                           P.desc.d, P.desc.ld, P.desc.M, im);
        return hipGetLastError();
    }
    const dim3 grid(static_cast<unsigned>((P.n_tiles + kAggQuads - 1) / kAggQuads));  // a tile per wave
    // Tiles of more segments than a wave takes one by one: the variant that
    // looks up every element's constant, derived once per (worker, segment)
    // by a launch of its own (16 quotients per thread and row otherwise).
    const int few_segs = agg_segs(P.desc.kind, P.level_bits, P.desc.M);
    const bool many = P.max_tile_segs > few_segs;
    if (many) {
        hipError_t err = launch_consts_from_scales(P, w.scale, st);
        if (err != hipSuccess) return err;
    }
    return with_dense_kind(P, [&](auto K, auto L) {
        if constexpr (decltype(K)::value == kIdentity) {
            return hipErrorInvalidValue;  // served above
        } else {
            auto go = [&](auto many_c) {
                hipLaunchKernelGGL((k_aggregate<decltype(K)::value, decltype(L)::value, decltype(many_c)::value>), grid,
                                   dim3(kBlock), 0, st, w.sign, w.level, w.scale, Qhat, P.d_consts, P.d_off,
                                   P.d_tile_seg, a, im, few_segs);
                return hipGetLastError();
            };
            return many ? go(std::true_type{}) : go(std::false_type{});
        }
    });
}

hipError_t launch_topk_apply(const dqgan_plan_s &P, float eta, const float *G, float *E, float *W, float *WX,
                             const dqgan_wire &w, float *Qhat, hipStream_t st) {
    const RowArgs a = row_args(P, eta, 0);
    return fused_by_m<kTopk, 0>(P, a, G, E, W, WX, w, Qhat, st);
}

hipError_t launch_topk_encode_rows(const dqgan_plan_s &P, float eta, const float *G, float *E, const dqgan_wire &w,
                                   hipStream_t st) {
    const RowArgs a = row_args(P, eta, 0);
    TopkArgs ta{P.topk.rows, P.topk.tile_off, P.topk.chunk_off, P.topk.n_tiles, P.topk.n_chunks, P.desc.k, w.idx};
    with_stream(worker_streams(P.desc), [&](auto S) {
        hipLaunchKernelGGL(k_topk_encode_rows<decltype(S)::value>,
                           dim3(static_cast<unsigned>(P.topk.n_tiles), static_cast<unsigned>(P.desc.M)), dim3(64), 0,
                           st, G, E, w.val, a, ta);
    });
    return hipGetLastError();
}

hipError_t launch_omd(const dqgan_plan_s &P, float eta, const float *Qhat, float *W, const float *G, const float *E,
                      float *WX, hipStream_t st) {
    with_stream(worker_streams(P.desc), [&](auto S) {
        hipLaunchKernelGGL(k_omd<decltype(S)::value>, dim3(static_cast<unsigned>(P.n_tiles)), dim3(kBlock), 0, st, Qhat,
                           W, G, E, WX, eta, P.desc.d, P.desc.ld, P.desc.M);
    });
    return hipGetLastError();
}

}  // namespace dq
