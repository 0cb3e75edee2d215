// Internal interface between the host ABI (capsule_host.cpp) and the HIP
// kernels (capsule_copy.hip, linattn_scan.hip, linattn_seg.hip,
// linattn_step.hip, gdn_scan.hip, gdn_step.hip, kv_fp8.hip, append.hip), and
// the rules that size their launches.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "capsule.h"

namespace cap {

// Launch a kernel whose one argument is a parameter struct passed by value
// and return that launch's own status.  The library never calls
// hipGetLastError, so an error the caller left pending is neither read nor
// cleared by a launch.
template <class P>
inline hipError_t launch_kernel(const void* fn, dim3 grid, dim3 block, const P& p, hipStream_t stream) {
    void* args[] = {const_cast<P*>(&p)};
    return hipLaunchKernel(fn, grid, block, args, 0, stream);
}

// One entry of a live set's static device segment table.  For buffer i of a
// set, with the boundary P' chosen per call:
//   capsule byte offset of buffer i = a + P' * b
// where a sums the bytes of the fixed buffers before i and b sums the
// row_bytes of the positional buffers before i.  Entry n (one past the last
// buffer) carries the totals, so the capsule size is a[n] + P' * b[n] and
// buffer i occupies [a[i] + P' b[i], a[i+1] + P' b[i+1]).  All values are
// multiples of 16 bytes.
struct SegEntry {
    uint64_t ptr;  // live device address of buffer i (0 in entry n)
    uint64_t a;
    uint64_t b;
};

constexpr int kMaxRep = 64;   // destination sets of a gather per launch
constexpr int kMaxDst = 16;   // destinations per source (fork)
constexpr int kMaxPtrLds = 2048;  // live pointers one copy block holds in LDS

enum CopyMode : int { kLiveToArena = 0, kArenaToLive = 1, kGather = 2 };

// Per-launch arguments of the copy kernel, passed by value.
//   kLiveToArena : rep 0 copies set `tabs[0]` -> arena_out.
//   kArenaToLive : rep r copies arena_in[r] -> n_dst destination sets
//                  tabs[r * n_dst + d] (fork: one rep, n_dst sets; a gather
//                  that stores little: n_rep reps, one set each).
//   kGather      : rep r copies arena_in[r] -> the sets tabs[first[r]] ..
//                  tabs[first[r + 1] - 1].
struct CopyParams {
    const SegEntry* layout;            // any table of the call (shared a, b)
    const SegEntry* tabs[kMaxRep];
    const uint8_t*  arena_in[kMaxRep];
    uint8_t*        arena_out;
    uint64_t        P;                 // aligned boundary
    uint64_t        nvec;              // capsule bytes / 16
    uint32_t        n_seg;
    uint32_t        n_dst;
    uint32_t        n_rep;
    int32_t         mode;
};

// A kGather launch.  `first` is an argument of that kernel only, so that the
// other copies do not pass it along.
struct GatherParams : CopyParams {
    uint8_t first[kMaxRep + 1];
};

// Whether a launch of a gather that stores `bytes` to each of n environments
// shares its reads between them.  Only above 128 MB, where the lookups per tile
// pay (us, destinations in turn, a rep to each environment / shared: 16
// environments of 2.4 MB 10.9 / 14.6, 40 of 1.2 MB 15.3 / 17.7, 31 of 3.5 MB 31.0 /
// 31.7, 24 of 4.7 MB, 113 MB in all, 33.5 / 34.8; 31 of 4.7 MB, 146 MB, 42.1 / 35.1,
// 16 of 9.4 MB 45.5 / 36.8, 64 of 4.7 MB 84.0 / 59.4).
constexpr uint64_t kGatherShareBytes = 128 << 20;
inline bool gather_shares(uint32_t n, uint64_t bytes) { return n * bytes > kGatherShareBytes; }
// Blocks a gather of the capsule p describes takes for each rep.
uint64_t gather_tiles(const CopyParams& p);
// Whether launch_copy accepts p (grid and LDS-table limits); a multi-launch
// call checks every launch with it before enqueueing the first one.
bool copy_params_ok(const CopyParams& p);
// Launch the descriptor-driven copy.  Returns hipSuccess or the launch error.
hipError_t launch_copy(const CopyParams& p, int num_cus, hipStream_t stream);
// The same for mode kGather.
hipError_t launch_gather(const GatherParams& p, hipStream_t stream);

// Placement of kernels that take a CU for each workgroup and in which the
// `per` workgroups of a head read the same lines.  Workgroups go round-robin
// over the 8 XCDs, each with an L2 of its own.  By XCD, XCD b % 8 takes all
// slices of an eighth of the heads, neighbouring ones (the XCDs differ by one
// head where 8 does not divide the head count, and the workgroups of the
// missing ones end at once); otherwise they are dealt out one by one.
// Measured (us, dealt / by XCD): delta-rule prefill of 4000 tokens x 128
// columns, 20 heads 126 / 113, 28 heads 143 / 115; linear-attention prefill of
// 900 tokens, 28 heads 28.2 / 22.9.  Not by XCD
//  * where the fullest XCD, of 32 CUs, would then need more rounds than the
//    deal: delta-rule prefill of 4000 tokens, 17 heads x 192 columns 113 / 198,
//    20 x 176 120 / 202; linear attention, 2048 tokens, 17 x 192 39.3 / 70.2;
//  * where it would have half as much again as its share (1 head, 900 tokens
//    with chunk states: 20.4 us, on one XCD 21.4; 10 heads x 256 columns, 300
//    tokens: 12.8 and 13.7);
//  * with one slice a head, where nothing is read twice (delta-rule prefill of 17
//    tokens, 12 heads x 16 columns: 11.5 and 11.8).
inline bool heads_by_xcd(int H, int per) {
    const int64_t most = (H + 7) / 8, dealt = ((int64_t)H * per + 7) / 8;  // heads, workgroups of the fullest XCD
    return H >= 8 && per > 1 && most * 16 <= 3 * (int64_t)H && (most * per + 31) / 32 <= (dealt + 31) / 32;
}
inline unsigned head_slice_grid(int H, int per) {
    return (unsigned)(heads_by_xcd(H, per) ? (H + 7) / 8 * 8 : H) * (unsigned)per;
}
// Rounds that the fullest XCD then needs.
inline int64_t scan_rounds(int H, int per) {
    const int64_t most = heads_by_xcd(H, per) ? (int64_t)((H + 7) / 8) * per : ((int64_t)H * per + 7) / 8;
    return (most + 31) / 32;
}
struct HeadSlice {
    int h, slice;
    bool on;
};
// (As one count `w` over heads and slices: computed for head and slice apart, the
// delta-rule scan keeps the scalars of its chunk loop in other registers and 4000
// tokens take 1 to 2 % longer.)
__host__ __device__ inline HeadSlice head_slice(unsigned b, bool by_xcd, int H, int per) {
    int w = (int)b, end = H * per;
    if (by_xcd) {
        const unsigned xcd = b % 8;
        w = (int)((uint64_t)xcd * (unsigned)H / 8) * per + (int)(b / 8);
        end = (int)((uint64_t)(xcd + 1) * (unsigned)H / 8) * per;
    }
    return {w / per, w % per, w < end};
}

// Scan arguments after host validation (sizes as 64-bit, pointers raw).
struct ScanParams {
    const void*  q;
    const void*  k;
    const void*  v;
    const float* g;
    const float* state_in;
    float*       o;
    float*       chunk_states;
    float*       final_state;
    int64_t      T;
    int32_t      H, dk, dv;
    int32_t      in_f32;   // 1: q/k/v are fp32, 0: bf16
    float        scale;
    int32_t      by_xcd;   // heads_by_xcd of the launch
};

// Host checks of a linattn_args (status codes as documented in capsule.h);
// on CAP_OK *out holds the launch parameters.
int validate_linattn(const linattn_args* a, ScanParams* out);

// A call in segments of G chunks (the last takes the rest), nseg of them;
// the second launch has a workgroup per segment, head and `cols` columns.
struct SegPlan {
    int64_t G, nseg;
    int cols;
};
constexpr int kSegWorkgroups = 512;  // two per CU (with fp32 inputs one fits: two rounds)
inline SegPlan linattn_seg_plan(const ScanParams& p) {
    const int64_t n = (p.T + 63) / 64;
    SegPlan s;
    // Columns per workgroup: 128 halve the reads of Q and K, 64 halve the time
    // of one chunk and give twice the workgroups.  16384 tokens x 16 heads (4096
    // workgroup-chunks of 128 columns): 153 us, with 64 columns 165; 2048 x 16
    // (512): 34 and 31.  The line between the two is not measured.
    s.cols = !p.in_f32 && p.dv > 64 && n * p.H * ((p.dv + 127) / 128) >= 3072 ? 128 : 64;
    // Segments: as many as run at once (more only add hand-over traffic:
    // 16384 x 32, 256 to 282 us with 2048 workgroups), each with at least the dk
    // tokens that its hand-over takes in o.
    const int64_t per = (int64_t)p.H * ((p.dv + s.cols - 1) / s.cols);
    const int64_t want = per < kSegWorkgroups ? kSegWorkgroups / per : 1;
    s.G = (n + want - 1) / want;
    if (!p.chunk_states && s.G < p.dk / 64) s.G = p.dk / 64;
    s.nseg = (n + s.G - 1) / s.G;
    if (!p.chunk_states && s.nseg > 1 && p.T - (s.nseg - 1) * s.G * 64 < p.dk) --s.nseg;
    return s;
}

// Whether a linear-attention prefill runs in segments of the sequence
// (linattn_seg.hip) or in one pass (linattn_scan.hip); both give the same bits.
// In chunks n and in x, 4 for each head and 64 columns begun: while the pass
// takes one round it takes 4.5 us + 0.98 us a chunk whatever x, the segments
// 11 us + a rate that grows with x.  Measured at up to 64 heads x 256 columns,
// inputs repeated and in turn (pass / segments, us; in brackets the lowest and
// highest ratio over all shapes at a number of chunks, bf16 and dk 128 where
// nothing is said):
//   x <= 64    1024 tokens x 8 heads x 128 columns 20.9 / 19.1 [16: 1.01 to 1.15];
//              dk 64 [16: 0.99 to 1.21]; fp32, 512 tokens [8: 1.04 to 1.12]
//   x <= 128   2048 x 16 x 128 37.7 / 31.4 [16: from 0.83, 28: from 1.00]; dk 64 [up
//              to x = 96, 28: from 0.96, 32: 1.03; beyond, 32: 0.96, 48: 1.04]; fp32
//              [32 heads x 64, 28 to 36: 0.97 to 1.00; else 28: 1.01]
//   x <= 144   [32: 0.88 to 1.14, 64: 1.01 to 1.40]; dk 64 [64: 1.07 to 1.15]
//   x <= 176   [64: 0.94 to 1.40, 96: 1.02 to 1.50]; dk 64 [64: 0.99 to 1.19, 128:
//              0.99 to 1.37]
//   x <= 256   8192 x 32 x 128 140 / 147, 8384 x 32 x 128 as long, 16384 x 32 288 / 260,
//              x 16 256 / 153 [96: 0.92 to 1.20, 130: from 1.00]; dk 64 [128: 0.93 to
//              1.21, 256: 1.01 to 1.40]
//   two rounds [up to x = 320, 32: 1.04 to 1.22; up to 384, 32: 0.94 to 1.10, 40: 1.03 to
//              1.21; beyond, 48: 0.95 to 1.13, 64: 1.00 to 1.23]; dk 64 [up to 384, 48:
//              1.00 to 1.23; beyond, 64: 0.95 to 1.19, 128: 1.07 to 1.30]
//   more       [32: 1.02 to 1.28]; dk 64 [32: 0.98 to 1.21, 48: 1.03 to 1.33]
// A last segment that takes `late` chunks more than the others (its own would
// hold fewer than the dk tokens of a hand-over in o) holds the call up: 981
// tokens x 6 heads x 16 columns 19.8 / 24.9; with five chunks more for each
// nothing measured loses.
// Never
//   * above x = 256 a round, where ragged widths leave segments half empty
//     columns: 2048 x 48 x 80 37 / 54, 4096 x 25 x 144 67 / 84;
//   * above x = 128 where the heads' placement (heads_by_xcd) would have to be
//     dealt out: 16384 x 18 x 176 [0.76 to 0.95, 1.00 once];
//   * above x = 128 with fp32 inputs (4096 x 32 x 128 86.6 / 99.1), whose second
//     kernel fits once on a CU, or with chunk states, where 32 heads fill the
//     chip either way (16384 x 32 350 / 356; fewer heads would gain there, up to
//     x = 176 [96: 1.04 to 1.70], up to 256 [96: 0.95 to 1.48], and do not take it).
inline bool linattn_in_segments(const ScanParams& p) {
    const int64_t n = (p.T + 63) / 64, x = (int64_t)p.H * ((p.dv + 63) / 64) * 4;
    if (n < 8) return false;
    const int per = p.dv / 16;
    const int64_t rounds = scan_rounds(p.H, per);
    const bool d64 = p.dk == 64 && !p.in_f32;
    int64_t from;
    if (x <= 64) {
        from = p.in_f32 ? 8 : 16;
    } else if (x <= 128) {
        from = x <= 96 ? (d64 ? 32 : 28) : d64 ? 48 : p.in_f32 ? 40 : 28;
    } else if (p.in_f32 || p.chunk_states || x > 256 * rounds) {
        return false;
    } else if (rounds > 1) {
        const bool more = rounds > 2;
        from = more || x <= 320 ? (d64 ? 48 : 32) : x <= 384 ? (d64 ? 48 : 40) : (d64 ? 96 : 64);
    } else if (p.H > 10 && per > 1 && !heads_by_xcd(p.H, per)) {
        return false;
    } else {
        from = x <= 144 ? 64 : x <= 176 ? (d64 ? 128 : 96) : (d64 ? 256 : 144);
    }
    const SegPlan s = linattn_seg_plan(p);
    const int64_t late = n - s.nseg * s.G;
    return n >= from + (late > 0 ? 5 * late : 0);
}

hipError_t launch_linattn_scan(const ScanParams& p, hipStream_t stream);
// the same call in segments of the sequence (T > 64), the same bits
hipError_t launch_linattn_seg(const ScanParams& p, hipStream_t stream);
// T == 1, bf16 inputs (a decode step); same contract as launch_linattn_scan
hipError_t launch_linattn_step(const ScanParams& p, hipStream_t stream);

// Gated delta-rule prefill (bf16 q/k/v, fp32 gates, write strengths and
// state).  ws holds one record of kGdnWsRecord bytes per chunk of 64 tokens
// and head ([n_chunks][H]), written by the first launch and read by the
// scan: the causal blocks of the chunk's (I + A)^-1 as bf16 hi/lo MFMA
// operands (6 blocks x 2 KiB, in the scan's lane order), then G log2(e) (64
// fp32, inclusive in-chunk log-gate sums) and beta (64 fp32).
constexpr int64_t kGdnWsTBytes = 6 * 2048;
constexpr int64_t kGdnWsTabOff = kGdnWsTBytes;
constexpr int64_t kGdnWsRecord = kGdnWsTabOff + 2 * 64 * 4;

struct GdnParams {
    const void*  q;
    const void*  k;
    const void*  v;
    const float* g;
    const float* beta;
    const float* state_in;
    float*       o;
    float*       chunk_states;
    float*       final_state;
    uint8_t*     ws;
    int64_t      T;
    int32_t      H, dk, dv;
    float        scale;
    int32_t      by_xcd;  // heads_by_xcd of the launch
};

// Host checks of a gdn_args; need_ws: the call reads args->workspace (a
// decode step does not).  On CAP_OK *out holds the launch parameters (ws =
// the caller's workspace, or NULL when need_ws is false).
int validate_gdn(const gdn_args* a, bool need_ws, GdnParams* out);

hipError_t launch_gdn(const GdnParams& p, hipStream_t stream);
// T == 1 (a decode step): one launch, no workspace use
hipError_t launch_gdn_step(const GdnParams& p, hipStream_t stream);

// FP8 (OCP E4M3) conversion of up to kFp8MaxSeg segments in one launch.
// Segment s converts n_groups[s] groups of 16 elements from src[s] to
// dst[s]; block b of the grid works on segment s with first_block[s] <= b <
// first_block[s + 1].  Quantize multiplies by mul[s] (1 / scale) before
// encoding; dequantize multiplies the decoded value by mul[s] (scale).
constexpr int kFp8MaxSeg = 64;
constexpr int kFp8GroupsPerBlock = 256;  // 256 threads x 2 units of 8 elements

// A launch counts its threads along x in 32 bits: 2^24 - 1 blocks of 256, which
// 6.9e10 elements pass (206 GB on both sides).  So block b is (b % kFp8GridX,
// b / kFp8GridX); the blocks past the last one find no elements.
constexpr uint32_t kFp8GridX = 1u << 22;
inline uint32_t fp8_grid_x(uint32_t blocks) { return blocks < kFp8GridX ? blocks : kFp8GridX; }
inline uint32_t fp8_grid_y(uint32_t blocks) { return (blocks + kFp8GridX - 1) / kFp8GridX; }

struct Fp8Params {
    uint64_t src[kFp8MaxSeg];
    uint64_t dst[kFp8MaxSeg];
    uint64_t n_groups[kFp8MaxSeg];
    uint32_t first_block[kFp8MaxSeg + 1];
    float    mul[kFp8MaxSeg];
    uint32_t n_seg;
    int32_t  quantize;  // 1: bf16 -> e4m3, 0: e4m3 -> bf16
};

hipError_t launch_fp8(const Fp8Params& p, hipStream_t stream);

// Append of a suffix of n tokens to a live set (one launch, up to
// kAppendMaxSeg buffers).  Segment s is either a positional copy of
// bytes[s] bytes from src[s] to dst[s] (tiles of kAppendTile bytes, several
// blocks), or, when win[s] != 0, a sliding window of win[s] bytes at dst[s]
// that takes the last win[s] bytes of (window, then the bytes[s] source
// bytes) in one block.  Block b works on segment s with first_block[s] <= b
// < first_block[s + 1].
constexpr int kAppendMaxSeg = 128;
constexpr uint32_t kAppendTile = 16384;        // bytes per positional block
constexpr uint32_t kAppendMaxWindow = 65536;   // bytes of one window

struct AppendParams {
    uint64_t src[kAppendMaxSeg];
    uint64_t dst[kAppendMaxSeg];
    uint64_t bytes[kAppendMaxSeg];
    uint32_t win[kAppendMaxSeg];
    uint32_t first_block[kAppendMaxSeg + 1];
    uint32_t n_seg;
};

hipError_t launch_append(const AppendParams& p, hipStream_t stream);

}  // namespace cap
