// Long calls of the chunked gated linear-attention prefill on gfx950, in
// segments of the sequence: the arithmetic of linattn_scan.hip, spread over
// the chip along the tokens too.
//
// For chunk j with entering state S_j (see linattn_scan.hip)
//   o_i     = scale * (exp(G_i) q_i S_j + sum_{m<=i} exp(G_i - G_m)(q_i.k_m) v_m)
//   S_{j+1} = exp(G_last) S_j + D_j,  D_j = sum_m exp(G_last - G_m) k_m^T v_m
// only S_{j+1} = exp(G_last) S_j + D_j is a true recurrence, one fma per
// element; D_j and the scores do not depend on S.  linattn_scan.hip walks all
// chunks with one workgroup per (head, 16 value columns): about 1 us a chunk
// however few heads there are, and every slice of a head reads the head's Q
// and K and forms its scores again.  Here a call is cut into segments of G
// chunks and runs as two launches:
//  1. linattn_fold: the states entering the segments, nothing else.
//  2. linattn_seg: one workgroup per (segment, head, 64 or 128 value columns)
//     walks the chunks of its segment from that state, forms the scores once
//     for all its columns, keeps its state in accumulator registers and writes
//     o, the chunk states and, in the last segment, the final state.
//
// The states between the launches need no memory of their own: they are left
// in chunk_states where the caller asked for them (entry c is the state
// entering chunk c) and otherwise in o, in the rows of the segment they
// enter: dk rows of dv floats, read back by the workgroup that later writes
// those rows, and by each wave only in the columns it writes itself.  So a
// segment has at least dk tokens.
//
// Bits.  A chunk's arithmetic depends only on (S_j, the chunk's inputs).
// Both kernels here use the operands, the order of every contraction and the
// fused multiply-adds of linattn_scan.hip, so neither the route nor the
// segments change a bit, and a call started at an aligned position from a
// restored state equals one longer call whichever way each of them runs.
//
// Measured (us, dk = dv = 128, final state only; linattn_scan.hip / this):
// 16384 tokens x 1 head 251 / 80, x 16 heads 256 / 153, x 32 heads 288 / 260;
// 2048 x 16 heads 37.7 / 31.4.  At 16384 x 32 a kernel trace gives the first
// launch 125 and the second 141 us.  The second moves 726 MB (counters; 709 are
// its inputs and outputs), 5.2 TB/s, with the MFMA pipe 25 % busy.  The first
// moves 337 MB; a workgroup asks the L2, which serves K to the eight of a head,
// for 293 lines a chunk (375 cycles on average), the texture address unit is
// busy 70 % of the time and a SIMD issues 39 %.
//
// Operand layouts.  The rows that a tile stands for are free:
//  * K^T of the fold is read with columns 32 (u / 2) + 8 (li / 4) + 4 (u % 2) +
//    li % 4 as row li of tile u, so that a lane's elements of the state tiles 2 kk
//    and 2 kk + 1 are d = 32 kk + 8 grp .. +7: as they lie in registers they are the
//    B operand of Q S with Q in its natural order;
//  * a score accumulator (K Q^T) holds P^T[16 mb + 4 grp + r][i], the A operand
//    of P V, handed to the other waves through LDS as such;
//  * with 128 columns a wave's two column tiles interleave (tile t, lane li:
//    column 2 li + t), so o and the states leave as 8-byte stores, a full
//    128-byte line per row and wave.
#include <hip/hip_runtime.h>
#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace cap {
namespace {

using namespace dev;

constexpr int CH = 64;  // chunk length

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

struct SegParams {
    ScanParams s;
    int32_t G;     // chunks per segment (the last segment takes the rest)
    int32_t nseg;
};

// an offset outside every buffer range, also with a chunk's or a state's
// offsets (below 2^31) added to it
constexpr uint32_t kOob = 0x7ffffff0u;

__device__ inline uint32_t chunk_rows(int64_t T, int64_t c) {
    const int64_t left = T - c * CH;
    return left >= CH ? (uint32_t)CH : (left > 0 ? (uint32_t)left : 0u);
}

// A per-lane offset the compiler recomputes where it is used instead of
// keeping one register per access over the whole loop.
__device__ inline uint32_t fresh(uint32_t x) {
    __asm__ volatile("" : "+v"(x));
    return x;
}

// The phases of a chunk stay apart in the schedule: hoisting one's LDS reads
// over another would not fit the registers two workgroups per CU leave.
__device__ inline void phase() { __builtin_amdgcn_sched_barrier(0); }

// Four fp32 elements as bf16 hi + lo, and the same of the elements times w.
// The products are rounded once for hi and enter lo exactly (one fma).
__device__ inline void split4(const u32x4& x, bf16x4& hi, bf16x4& lo) {
    const f32x4 a = __builtin_bit_cast(f32x4, x);
    const float f[4] = {a[0], a[1], a[2], a[3]};
    split_n<4>(f, hi, lo);
}

__device__ inline void split4w(const u32x4& x, float w, bf16x4& hi, bf16x4& lo) {
    const f32x4 a = __builtin_bit_cast(f32x4, x);
    const float f[4] = {a[0], a[1], a[2], a[3]}, ww[4] = {w, w, w, w};
    split_product<4>(f, ww, hi, lo);
}

// V w as MFMA operands from a V operand (8 exact bf16) and its rows' weights.
__device__ inline void weigh(const bf16x8& v, const f32x4& w0, const f32x4& w1, bf16x8& hi, bf16x8& lo) {
    float f[8], w[8];
    #pragma unroll
    for (int e = 0; e < 4; ++e) {
        f[e] = (float)v[e];
        f[4 + e] = (float)v[4 + e];
        w[e] = w0[e];
        w[4 + e] = w1[e];
    }
    split_product<8>(f, w, hi, lo);
}

// Operands whose contraction index runs along the rows of an LDS tile; lane li
// is column n0 + li.  trn: k-slot 8 grp + e is row k0 + 8 grp + e; tra: row k0 +
// 16 (e / 4) + 4 grp + e % 4, the order in which two accumulators hold their
// rows.
__device__ inline bf16x8 trn(const __bf16* tile, int pitch, int k0, int n0, int li, int grp) {
    return cat(tr4(tile, pitch, k0 + 8 * grp, n0, li), tr4(tile, pitch, k0 + 8 * grp + 4, n0, li));
}
__device__ inline bf16x8 tra(const __bf16* tile, int pitch, int k0, int n0, int li, int grp) {
    return cat(tr4(tile, pitch, k0 + 4 * grp, n0, li), tr4(tile, pitch, k0 + 16 + 4 * grp, n0, li));
}

// K^T for the fold: k-slot 8 grp + e is row k0 + 8 grp + e; row li of the operand
// is column 32 (u / 2) + 8 (li / 4) + 4 (u % 2) + li % 4, so that the state tiles 2 kk
// and 2 kk + 1 together hold d = 32 kk + 8 grp .. +7 per lane, the order of Q.
__device__ inline bf16x8 trk(const __bf16* tile, int pitch, int k0, int u, int li, int grp) {
    const __bf16* a = tile + (k0 + 8 * grp + (li >> 2)) * pitch + 32 * (u >> 1) + 8 * (li & 3) + 4 * (u & 1);
    const i16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)a);
    const i16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4*)(a + 4 * pitch));
    return cat(__builtin_bit_cast(bf16x4, x), __builtin_bit_cast(bf16x4, y));
}

// ------------------------------------------------------------------- fold
// A workgroup keeps DA rows x 16 columns of one head's state and takes eight
// chunks a round, a chunk per wave: the wave forms D = K^T (V w) of its chunk
// and hands it over in LDS; after the round's one barrier every thread runs
// the fma chain of its elements over the round's chunks while its wave already
// works on the next round (D is double buffered).  A round takes about 2 us
// on an idle chip, vector arithmetic, LDS and a load's latency in turn, and 4.2
// us (10,000 cycles; a wave issues 267 vector instructions in it, 32 of them
// MFMA of 16 cycles) when 256 workgroups share the L2.
//
// K never passes through LDS: lane (li, grp) loads columns NU li .. +NU - 1 of
// the rows 32 mm + 8 grp + e, so each load takes whole rows of the head, and
// pairs of its registers, half-words exchanged, are operands: tile t then
// stands for the rows d = NU li + t of the state.  (K through LDS and the
// transposing load took as long, with three times the LDS traffic.)  Loads are
// two rounds ahead, in two register stages.
constexpr int kFoldWaves = 8;     // chunks in progress per workgroup
constexpr int kFoldPrefetch = 3;  // rounds the L2 prefetch is ahead

template <int DA, bool F32>
struct alignas(16) FoldSmem {
    static constexpr int NW = kFoldWaves, NP = F32 ? 2 : 1;
    alignas(16) __bf16 v[NW][NP][CH * 16];   // bf16: V; fp32 inputs: V w hi, lo
    alignas(16) float w[NW][CH];
    alignas(16) float d[2][NW][DA * 16];     // D [d][16], by round parity
    float gamma[2][NW];
};

template <int DK, int DA, bool F32>
__global__ __launch_bounds__(64 * kFoldWaves, 2) void linattn_fold_kernel(const SegParams sp) {
    using Sm = FoldSmem<DA, F32>;
    constexpr int NW = Sm::NW, NP = Sm::NP;
    constexpr int DB = DK / DA, NU = DA / 16;        // row blocks of the state, tiles of 16 rows in one
    constexpr bool PF = DA == 128;
    constexpr int ES = F32 ? 4 : 2, EPP = 16 / ES;   // bytes per element, elements per 16-byte piece
    constexpr int KD = NU * ES / 4;                  // dwords of a K row per lane
    constexpr int VPR = 16 / EPP, VR = 64 / VPR, NV = CH / VR;
    __shared__ Sm sm;
    const ScanParams& p = sp.s;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = p.H, dv = p.dv;

    // workgroup -> (head, row block, columns)
    const int per = DB * (dv / 16);
    const HeadSlice hs = head_slice(blockIdx.x, p.by_xcd, H, per);
    if (!hs.on) return;
    const int h = hs.h, slice = hs.slice;
    const int d0 = DA * (slice % DB), j0 = 16 * (slice / DB);
    const int64_t qk_row = (int64_t)H * DK * ES, v_row = (int64_t)H * dv * ES;
    const int nA = (sp.nseg - 1) * sp.G;             // chunks to fold, all full

    // D granules (16 bytes) of a row are swizzled by row: the rows that one
    // access serves together lie in different banks
    auto dpos = [](int row, int j4) { return row * 16 + ((j4 ^ ((row / NU ^ row) & 3)) << 2); };

    // ---- loads of one chunk: row e of half operand mm, V pieces, gates
    struct Stage {
        uint32_t k[2][8][KD];
        u32x4 v[NV];
        float g;
    };
    const uint32_t koff = (uint32_t)(8 * grp * qk_row + ((int64_t)h * DK + d0 + NU * li) * ES);
    const int vrow = lane / VPR, vcol = EPP * (lane % VPR);
    const uint32_t voff = (uint32_t)(vrow * v_row + ((int64_t)h * dv + j0 + vcol) * ES);
    auto load_k = [&](Stage& R, int c, int mm) __attribute__((always_inline)) {
        const rsrc_t rk = make_rsrc_u32(static_cast<const char*>(p.k) + (int64_t)c * CH * qk_row,
                                        c < nA ? CH * (uint32_t)qk_row : 0u);
        #pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t off = koff + (uint32_t)(32 * mm + e) * (uint32_t)qk_row;
            if constexpr (KD == 4) {
                const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(rk, off, 0, 0);
                #pragma unroll
                for (int y = 0; y < KD; ++y) R.k[mm][e][y] = x[y];
            } else {
                const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(rk, off, 0, 0);
                R.k[mm][e][0] = x[0];
                R.k[mm][e][1] = x[1];
            }
        }
    };
    auto load_vg = [&](Stage& R, int c) __attribute__((always_inline)) {
        const uint32_t rows = c < nA ? (uint32_t)CH : 0u;
        const rsrc_t rv = make_rsrc_u32(static_cast<const char*>(p.v) + (int64_t)c * CH * v_row, rows * (uint32_t)v_row);
        const rsrc_t rg = make_rsrc_u32(p.g + (int64_t)c * CH * H, rows * (uint32_t)(H * 4));
        R.g = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, (uint32_t)((lane * H + h) * 4), 0, 0));
        #pragma unroll
        for (int i = 0; i < NV; ++i)
            R.v[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, voff + (uint32_t)(VR * i) * (uint32_t)v_row, 0, 0);
    };

    // ---- the chain: this thread's elements of the state, four columns each
    constexpr int CT = DA * 4;
    constexpr int NE = (CT + 64 * NW - 1) / (64 * NW);
    static_assert(NE == 1, "one quad per thread");
    const int dd = (tid >> 2) & (DA - 1), jq = tid & 3;
    const bool on = tid < CT;
    f32x4 S = {0.f, 0.f, 0.f, 0.f};
    if (on && p.state_in) S = *reinterpret_cast<const f32x4*>(p.state_in + ((int64_t)h * DK + d0 + dd) * dv + j0 + 4 * jq);
    // the states entering the segments, left in chunk_states or in o
    const int64_t step = p.chunk_states ? (int64_t)sp.G * H * DK * dv : (int64_t)sp.G * CH * H * dv;
    float* dst = p.chunk_states ? p.chunk_states + ((int64_t)h * DK + d0 + dd) * dv + j0 + 4 * jq
                                : p.o + ((int64_t)(d0 + dd) * H + h) * dv + j0 + 4 * jq;
    auto park = [&]() __attribute__((always_inline)) {
        if (on) *reinterpret_cast<f32x4*>(dst) = S;
        dst += step;
    };
    int next = 0;  // the next segment's first chunk

    // Cooperative L2 prefetch.  A head's workgroups read the same K lines and
    // share those of V and g; missed by all of them at the same moment, a line
    // costs each a full HBM latency.  So every workgroup touches its share of
    // the lines (K, then V, then g; line x goes to workgroup x % per) ahead of
    // the loads, which then hit in L2.  The word read is only consumed as an
    // asm operand two rounds later, forcing nothing but the load's completion.
    // Only with the whole row block in one workgroup, the shape of calls that
    // fill the chip (a call of 16384 tokens x 32 heads 272 -> 257 us, x 24 229 ->
    // 214); with fewer workgroups the misses overlap anyway and it costs 1 to 3 %.
    uint32_t pf[2] = {0u, 0u};
    const char* pbase = static_cast<const char*>(p.k);
    int64_t prow = 0;  // bytes per token of the lane's line, 0: no line
    if constexpr (PF) {
        constexpr int LK = DK * ES / 128;
        const int LV = (dv * ES + 127) / 128, x = slice + per * lane;
        if (x < CH * LK) {
            prow = qk_row;
            pbase += (int64_t)(x / LK) * qk_row + (int64_t)h * DK * ES + (x % LK) * 128;
        } else if (x < CH * (LK + LV)) {
            const int y = x - CH * LK;
            prow = v_row;
            pbase = static_cast<const char*>(p.v) + (int64_t)(y / LV) * v_row + (int64_t)h * dv * ES + (y % LV) * 128;
        } else if (x < CH * (LK + LV + 1)) {
            prow = (int64_t)H * 4;
            pbase = reinterpret_cast<const char*>(p.g) + (int64_t)(x - CH * (LK + LV)) * prow + h * 4;
        }
    }
    auto prefetch = [&](int slot, int c) __attribute__((always_inline)) {
        if constexpr (!PF) return;
        __asm__ volatile("" : : "v"(pf[slot]));
        pf[slot] = *reinterpret_cast<const uint32_t*>(pbase + (c < nA ? (int64_t)c * CH * prow : 0));
    };
    // one round: the chunks cb .. cb + NW - 1, this wave's in R, which then
    // takes its chunk two rounds on
    auto round = [&](int cb, int b, Stage& R) __attribute__((always_inline)) {
        prefetch(b, cb + kFoldPrefetch * NW + wave);
        // weights and V into this wave's LDS
        const float xs = wave_inclusive_sum(R.g);
        const float glast = lane_value(xs, 63);
        const float wl = __expf(glast - xs);
        sm.w[wave][lane] = wl;
        sm.gamma[b][wave] = __expf(glast);
        #pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = VR * i + vrow, at = row * 16 + vcol;
            if constexpr (F32) {
                bf16x4 hi, lo;
                split4w(R.v[i], __shfl(wl, row, 64), hi, lo);
                *reinterpret_cast<bf16x4*>(&sm.v[wave][0][at]) = hi;
                *reinterpret_cast<bf16x4*>(&sm.v[wave][NP - 1][at]) = lo;
            } else {
                *reinterpret_cast<u32x4*>(&sm.v[wave][0][at]) = R.v[i];
            }
        }
        phase();
        load_vg(R, cb + 2 * NW + wave);
        phase();
        // D, transposed in the accumulators: lane (li, grp) of tile t holds
        // D[NU li + t][4 grp .. +3]
        f32x4 D[NU];
        #pragma unroll
        for (int t = 0; t < NU; ++t) D[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
            bf16x8 wh, wlo;
            if constexpr (F32) {
                wh = trn(sm.v[wave][0], 16, 32 * mm, 0, li, grp);
                wlo = trn(sm.v[wave][NP - 1], 16, 32 * mm, 0, li, grp);
            } else {
                const f32x4 w0 = *reinterpret_cast<const f32x4*>(&sm.w[wave][32 * mm + 8 * grp]);
                const f32x4 w1 = *reinterpret_cast<const f32x4*>(&sm.w[wave][32 * mm + 8 * grp + 4]);
                weigh(trn(sm.v[wave][0], 16, 32 * mm, 0, li, grp), w0, w1, wh, wlo);
            }
            #pragma unroll
            for (int t = 0; t < NU; ++t) {
                bf16x8 kh, kl;
                if constexpr (F32) {
                    float f[8];
                    #pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = __builtin_bit_cast(float, R.k[mm][e][t]);
                    split_n<8>(f, kh, kl);
                } else {
                    u32x4 x;
                    #pragma unroll
                    for (int y = 0; y < 4; ++y)
                        x[y] = __builtin_amdgcn_perm(R.k[mm][2 * y + 1][t >> 1], R.k[mm][2 * y][t >> 1],
                                                     (t & 1) ? 0x07060302u : 0x05040100u);
                    kh = __builtin_bit_cast(bf16x8, x);
                }
                D[t] = mma(wh, kh, D[t]);
                D[t] = mma(wlo, kh, D[t]);
                if (F32) D[t] = mma(wh, kl, D[t]);
            }
            phase();
            load_k(R, cb + 2 * NW + wave, mm);
            phase();
        }
        #pragma unroll
        for (int t = 0; t < NU; ++t)
            *static_cast<f32x4*>(__builtin_assume_aligned(&sm.d[b][wave][dpos(NU * li + t, grp)], 16)) = D[t];
        lds_barrier();
        // the chain over the round's chunks
        f32x4 Dc[NW];
        float gm[NW];
        #pragma unroll
        for (int x = 0; x < NW; ++x) {
            gm[x] = sm.gamma[b][x];
            Dc[x] = *reinterpret_cast<const f32x4*>(&sm.d[b][x][dpos(dd, jq)]);
        }
        #pragma unroll
        for (int x = 0; x < NW; ++x) {
            const bool live = cb + x < nA;  // wave-uniform
            if (live && cb + x == next) {
                park();
                next += sp.G;
            }
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float y = __builtin_fmaf(gm[x], S[r], Dc[x][r]);
                S[r] = live ? y : S[r];
            }
        }
    };
    Stage R0, R1;
    // in the order of the loop's loads: the compiler's in-order counters then
    // never wait for the younger stage
    load_vg(R0, wave);
    phase();
    load_k(R0, wave, 0);
    phase();
    load_k(R0, wave, 1);
    phase();
    load_vg(R1, NW + wave);
    phase();
    load_k(R1, NW + wave, 0);
    phase();
    load_k(R1, NW + wave, 1);
    phase();
    for (int cb = 0;;) {
        round(cb, 0, R0);
        if ((cb += NW) >= nA) break;
        round(cb, 1, R1);
        if ((cb += NW) >= nA) break;
    }
    park();  // the last segment's
    __asm__ volatile("" : : "v"(pf[0]), "v"(pf[1]));
}

// ---------------------------------------------------------------- segment
template <int DK, bool F32, int NT>
struct alignas(16) SegSmem {
    static constexpr int NL = F32 ? 2 : 1;
    static constexpr int KP = DK == 128 ? 160 : 96;  // pitch of K [m][d]
    static constexpr int QP = DK + 16;         // pitch of Q [i][d]
    static constexpr int VP = 64 * NT + 16;    // pitch of V [m][column]
    alignas(16) __bf16 k[NL][CH * KP];
    alignas(16) __bf16 q[NL][CH * QP];
    alignas(16) __bf16 v[NL][CH * VP];
    alignas(16) __bf16 vw[F32 ? 2 : 1][F32 ? CH * VP : 8];  // fp32 inputs: V w
    alignas(16) __bf16 p[6][2][512];           // decayed scores as operands: unit, hi / lo, lane
    alignas(16) float G2[2][CH];               // G_t log2(e), by chunk parity
    alignas(16) float eG[2][CH];               // exp(G_t)
    alignas(16) float w[2][CH];                // exp(G_last - G_t)
    alignas(16) float bm[2][CH];               // exp(G_e - G_m), e = last token of m's block of 16
    alignas(16) float ai[2][CH][4];            // exp(G_i - G_e(M)) for the blocks M before i's
};

// K rows: a pitch of 16 banks' dwords modulo 64 leaves the two-way conflict
// that the 8-byte pieces of trk have anyway; Q and V rows: 8, none.
//
// Two barriers a chunk.  Before the first the chunk's K, Q and V go from the
// registers they were loaded into a chunk earlier to LDS; between the two
// every wave forms its part of the scores (6 units of 16 rows x 32 tokens),
// then Q S and the fold for its own columns; after the second, P V and o.
// Two workgroups share a CU, so one computes while the other waits; a chunk of
// 128 columns takes one alone about 4.5 us.  That leaves 256 registers a wave
// (state 64, next chunk's loads 48, products 64): the column tiles are folded
// one after the other, the phases are kept apart in the schedule and offsets
// are recomputed, because a spilled load would be waited for where it is
// issued.
template <int DK, bool F32, int NT, bool CS>
__global__ __launch_bounds__(256, F32 ? 1 : 2) void linattn_seg_kernel(const SegParams sp) {
    using Sm = SegSmem<DK, F32, NT>;
    constexpr int KP = Sm::KP, QP = Sm::QP, VP = Sm::VP, NL = Sm::NL;
    constexpr int ES = F32 ? 4 : 2, EPP = 16 / ES;
    constexpr int NKK = DK / 32, NU = DK / 16;
    constexpr int KPR = DK / EPP, KR = 256 / KPR, NK = CH / KR;   // pieces per row, rows per load, loads
    constexpr int VPR = 64 * NT / EPP, VR = 256 / VPR, NV = CH / VR;
    static_assert(!(F32 && NT == 2), "fp32 inputs use one column tile per wave");
    __shared__ Sm sm;
    const ScanParams& p = sp.s;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int H = p.H, dv = p.dv;

    // segments from the last to the first, so that the K and V the first
    // launch read last are read first, from the Infinity Cache
    const int ncg = (dv + 64 * NT - 1) / (64 * NT);
    const int seg = sp.nseg - 1 - (int)(blockIdx.x / (unsigned)(H * ncg));
    const int rem = (int)(blockIdx.x % (unsigned)(H * ncg));
    const int h = rem % H, cg = rem / H;
    const int64_t n = (p.T + CH - 1) / CH;
    const int64_t c0 = (int64_t)seg * sp.G;
    const bool last_seg = seg == sp.nseg - 1;
    const int64_t c1 = last_seg ? n : c0 + sp.G;
    const int64_t qk_row = (int64_t)H * DK * ES, v_row = (int64_t)H * dv * ES, o_row = (int64_t)H * dv * 4;

    const int jw = 64 * NT * cg + 16 * NT * wave;      // the wave's first column
    const int jl = jw + NT * li;                       // the lane's first column (of NT)
    const bool jok = jl < dv;

    // ---- the state entering the segment: S[u][t][r] = S[32 (u / 2) + 8 grp + 4 (u % 2) + r][jl + t]
    f32x4 S[NU][NT];
    {
        const float* src = nullptr;
        int64_t stride = dv;
        if (sp.nseg == 1) {
            if (p.state_in) src = p.state_in + (int64_t)h * DK * dv;
        } else if (p.chunk_states) {
            src = p.chunk_states + (c0 * H + h) * DK * dv;
        } else {
            src = p.o + (c0 * CH * H + h) * dv;
            stride = (int64_t)H * dv;
        }
        // no state: an empty range (zeros); a lane without a column reads
        // another's, its columns are never stored
        const rsrc_t rs = make_rsrc_u32(src, src ? (uint32_t)((stride * (DK - 1) + dv) * 4) : 0u);
        const uint32_t so = (uint32_t)((8 * grp * stride + (jok ? jl : 0)) * 4);
        #pragma unroll
        for (int u = 0; u < NU; ++u)
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t off = so + (uint32_t)(32 * (u >> 1) + 4 * (u & 1) + r) * (uint32_t)(stride * 4);
                if constexpr (NT == 2) {
                    const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
                    const uint32_t x0 = x[0], x1 = x[1];
                    S[u][0][r] = __builtin_bit_cast(float, x0);
                    S[u][NT - 1][r] = __builtin_bit_cast(float, x1);
                } else {
                    S[u][0][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0));
                }
            }
    }

    // ---- loads of one chunk, coalesced
    u32x4 kr[NK], qr[NK], vr[NV];
    auto load = [&](int64_t c) {
        const int64_t t0 = c * CH;
        const uint32_t rows = c < c1 ? chunk_rows(p.T, c) : 0u;
        const rsrc_t rk = make_rsrc_u32(static_cast<const char*>(p.k) + t0 * qk_row, rows * (uint32_t)qk_row);
        const rsrc_t rq = make_rsrc_u32(static_cast<const char*>(p.q) + t0 * qk_row, rows * (uint32_t)qk_row);
        const rsrc_t rv = make_rsrc_u32(static_cast<const char*>(p.v) + t0 * v_row, rows * (uint32_t)v_row);
        const uint32_t tid = fresh(threadIdx.x);
        const uint32_t vcol = 64 * NT * cg + EPP * (tid % VPR);
        const uint32_t ko = (tid / KPR) * (uint32_t)qk_row + (uint32_t)(h * DK * ES) + (tid % KPR) * 16;
        const uint32_t vo = vcol < (uint32_t)dv ? (tid / VPR) * (uint32_t)v_row + ((uint32_t)(h * dv) + vcol) * ES : kOob;
        #pragma unroll
        for (int i = 0; i < NK; ++i)
            kr[i] = __builtin_amdgcn_raw_buffer_load_b128(rk, ko + (uint32_t)(KR * i) * (uint32_t)qk_row, 0, 0);
        #pragma unroll
        for (int i = 0; i < NK; ++i)
            qr[i] = __builtin_amdgcn_raw_buffer_load_b128(rq, ko + (uint32_t)(KR * i) * (uint32_t)qk_row, 0, 0);
        #pragma unroll
        for (int i = 0; i < NV; ++i)
            vr[i] = __builtin_amdgcn_raw_buffer_load_b128(rv, vo + (uint32_t)(VR * i) * (uint32_t)v_row, 0, 0);
    };
    // the gate wave (3, with one unit of the scores) alone reads the gates,
    // two chunks ahead, and writes the tables one chunk ahead
    float gr = 0.0f;
    auto load_g = [&](int64_t c) {
        if (wave != 3) return;
        const rsrc_t rg = make_rsrc_u32(p.g + c * CH * H, c < c1 ? chunk_rows(p.T, c) * (uint32_t)(H * 4) : 0u);
        gr = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, (uint32_t)((lane * H + h) * 4), 0, 0));
    };
    auto tables = [&](int b) {
        if (wave != 3) return;
        const int lane = (int)fresh((uint32_t)tid) & 63;
        const float xs = wave_inclusive_sum(gr);
        const float glast = lane_value(xs, 63);
        sm.w[b][lane] = __expf(glast - xs);
        sm.G2[b][lane] = xs * LOG2E;
        sm.eG[b][lane] = __expf(xs);
        float ge[4];
        #pragma unroll
        for (int M = 0; M < 4; ++M) ge[M] = lane_value(xs, 16 * M + 15);
        const int blk = lane >> 4;
        const float gb = blk == 0 ? ge[0] : blk == 1 ? ge[1] : blk == 2 ? ge[2] : ge[3];
        sm.bm[b][lane] = __expf(gb - xs);
        f32x4 a;
        #pragma unroll
        for (int M = 0; M < 4; ++M) a[M] = (M < blk) ? __expf(xs - ge[M]) : 0.0f;
        *reinterpret_cast<f32x4*>(&sm.ai[b][lane][0]) = a;
    };

    auto stage = [&](int b) {
        const int tid = (int)fresh(threadIdx.x);
        const int kcol = EPP * (tid % KPR), krow = tid / KPR, vloc = EPP * (tid % VPR), vrow = tid / VPR;
        #pragma unroll
        for (int i = 0; i < NK; ++i) {
            const int row = KR * i + krow;
            if constexpr (F32) {
                bf16x4 hi, lo;
                split4(kr[i], hi, lo);
                *reinterpret_cast<bf16x4*>(&sm.k[0][row * KP + kcol]) = hi;
                *reinterpret_cast<bf16x4*>(&sm.k[NL - 1][row * KP + kcol]) = lo;
                split4(qr[i], hi, lo);
                *reinterpret_cast<bf16x4*>(&sm.q[0][row * QP + kcol]) = hi;
                *reinterpret_cast<bf16x4*>(&sm.q[NL - 1][row * QP + kcol]) = lo;
            } else {
                *reinterpret_cast<u32x4*>(&sm.k[0][row * KP + kcol]) = kr[i];
                *reinterpret_cast<u32x4*>(&sm.q[0][row * QP + kcol]) = qr[i];
            }
        }
        #pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int row = VR * i + vrow;
            if constexpr (F32) {
                bf16x4 hi, lo;
                split4(vr[i], hi, lo);
                *reinterpret_cast<bf16x4*>(&sm.v[0][row * VP + vloc]) = hi;
                *reinterpret_cast<bf16x4*>(&sm.v[NL - 1][row * VP + vloc]) = lo;
                split4w(vr[i], sm.w[b][row], hi, lo);
                *reinterpret_cast<bf16x4*>(&sm.vw[0][row * VP + vloc]) = hi;
                *reinterpret_cast<bf16x4*>(&sm.vw[F32 ? 1 : 0][row * VP + vloc]) = lo;
            } else if constexpr (NT == 2) {
                // columns 2 x to tile 0 and 2 x + 1 to tile 1 of each 32
                const uint32_t a0 = vr[i][0], a1 = vr[i][1], a2 = vr[i][2], a3 = vr[i][3];
                const int at = row * VP + (vloc & ~31) + ((vloc & 31) >> 1);
                *reinterpret_cast<u32x2*>(&sm.v[0][at]) =
                    u32x2{__builtin_amdgcn_perm(a1, a0, 0x05040100u), __builtin_amdgcn_perm(a3, a2, 0x05040100u)};
                *reinterpret_cast<u32x2*>(&sm.v[0][at + 16]) =
                    u32x2{__builtin_amdgcn_perm(a1, a0, 0x07060302u), __builtin_amdgcn_perm(a3, a2, 0x07060302u)};
            } else {
                *reinterpret_cast<u32x4*>(&sm.v[0][row * VP + vloc]) = vr[i];
            }
        }
    };

    // ---- scores of rows 16 W .. +15 against tokens 32 pr .. +31, decayed, as
    // the A operand of P V: unit W for W < 2, else 2 W - 2 + pr
    auto score_unit = [&](int b, int unit) {
        const int W = unit < 2 ? unit : 1 + (unit >> 1), pr = unit < 2 ? 0 : (unit & 1);
        const int lane = (int)fresh((uint32_t)tid) & 63, li = lane & 15, grp = lane >> 4;
        bf16x8 qh[NKK], ql[NKK];
        const int qo = (16 * W + li) * QP + 8 * grp;
        #pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            qh[kk] = *reinterpret_cast<const bf16x8*>(&sm.q[0][qo + 32 * kk]);
            if (F32) ql[kk] = *reinterpret_cast<const bf16x8*>(&sm.q[NL - 1][qo + 32 * kk]);
        }
        const int i = 16 * W + li;
        const float gi = sm.G2[b][i];
        float f[8], w[8];
        #pragma unroll
        for (int half = 0; half < 2; ++half) {
            phase();
            const int m0 = 32 * pr + 16 * half;
            f32x4 at = {0.f, 0.f, 0.f, 0.f};
            if (m0 <= 16 * W) {  // wave-uniform; blocks above the diagonal are zero
                #pragma unroll
                for (int kk = 0; kk < NKK; ++kk) {
                    const int ko = (m0 + li) * KP + 32 * kk + 8 * grp;
                    const bf16x8 kh = *reinterpret_cast<const bf16x8*>(&sm.k[0][ko]);
                    at = mma(kh, qh[kk], at);
                    if (F32) {
                        at = mma(kh, ql[kk], at);
                        at = mma(*reinterpret_cast<const bf16x8*>(&sm.k[NL - 1][ko]), qh[kk], at);
                    }
                }
            }
            // decay: factored tables below the diagonal block, exp2 on it
            if (m0 < 16 * W) {
                const float ai = sm.ai[b][i][m0 >> 4];
                const f32x4 bmv = *reinterpret_cast<const f32x4*>(&sm.bm[b][m0 + 4 * grp]);
                #pragma unroll
                for (int r = 0; r < 4; ++r) {
                    f[4 * half + r] = at[r] * ai;
                    w[4 * half + r] = bmv[r];
                }
            } else {
                const f32x4 gm = *reinterpret_cast<const f32x4*>(&sm.G2[b][m0 + 4 * grp]);
                #pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = at[r] * __builtin_amdgcn_exp2f(gi - gm[r]);
                    f[4 * half + r] = (m0 + 4 * grp + r <= i) ? x : 0.0f;
                    w[4 * half + r] = 1.0f;
                }
            }
        }
        bf16x8 ph, pl;
        split_product<8>(f, w, ph, pl);
        *reinterpret_cast<bf16x8*>(&sm.p[unit][0][8 * lane]) = ph;
        *reinterpret_cast<bf16x8*>(&sm.p[unit][1][8 * lane]) = pl;
    };

    const uint32_t soff = jok ? (uint32_t)((((int64_t)h * DK + 8 * grp) * dv + jl) * 4) : kOob;
    const uint32_t ooff = jok ? (uint32_t)(4 * grp * o_row + ((int64_t)h * dv + jl) * 4) : kOob;
    auto chunk = [&](int64_t c, auto fold) {
        const int b = (int)(c & 1);
        stage(b);
        phase();
        if constexpr (fold.value) load(c + 1);
        lds_barrier();
        phase();

        tables(b ^ 1);
        load_g(c + 2);
        // wave 0: units 4 and 0, wave 1: 5, wave 2: 2 and 3, wave 3: 1 -- that is
        // 3, 2, 3 and 2 blocks of 16 x 16
        #pragma unroll 1
        for (int x = 0; x <= 1 - (wave & 1); ++x) score_unit(b, ((x ? 0x0300 : 0x1254) >> (4 * wave)) & 7);

        phase();
        // X = Q S; lane: row 16 rb + 4 grp + r, column jl + t
        f32x4 acc[NT][4], accl[NT][4];  // hi and lo products
        #pragma unroll
        for (int t = 0; t < NT; ++t)
            #pragma unroll
            for (int rb = 0; rb < 4; ++rb) acc[t][rb] = accl[t][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
        #pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
            if (kk > 0 && (NT == 2 || kk % 2 == 0)) phase();
            bf16x8 qh[4], ql[4];
            #pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                const int at = (16 * rb + li) * QP + 32 * kk + 8 * grp;
                qh[rb] = *reinterpret_cast<const bf16x8*>(&sm.q[0][at]);
                if (F32) ql[rb] = *reinterpret_cast<const bf16x8*>(&sm.q[NL - 1][at]);
            }
            #pragma unroll
            for (int t = 0; t < NT; ++t) {
                float f[8];
                #pragma unroll
                for (int r = 0; r < 4; ++r) {
                    f[r] = S[2 * kk][t][r];
                    f[4 + r] = S[2 * kk + 1][t][r];
                }
                bf16x8 sh, sl;
                split_n<8>(f, sh, sl);
                #pragma unroll
                for (int rb = 0; rb < 4; ++rb) {
                    acc[t][rb] = mma(qh[rb], sh, acc[t][rb]);
                    accl[t][rb] = mma(qh[rb], sl, accl[t][rb]);
                    if (F32) accl[t][rb] = mma(ql[rb], sh, accl[t][rb]);
                }
            }
        }
        #pragma unroll
        for (int t = 0; t < NT; ++t)
            #pragma unroll
            for (int rb = 0; rb < 4; ++rb) acc[t][rb] += accl[t][rb];

        phase();
        // the state entering the chunk, as chunk state c (the first launch wrote
        // the segment's first)
        if constexpr (CS) {
            const rsrc_t rc = make_rsrc_u32(p.chunk_states + c * (int64_t)H * DK * dv, c > c0 ? (uint32_t)(H * DK * dv * 4) : 0u);
            const uint32_t so = fresh(soff);
            #pragma unroll
            for (int u = 0; u < NU; ++u)
                #pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const uint32_t off = so + (uint32_t)(32 * (u >> 1) + 4 * (u & 1) + r) * (uint32_t)(dv * 4);
                    if constexpr (NT == 2) {
                        const f32x2 x = {S[u][0][r], S[u][NT - 1][r]};
                        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), rc, off, 0, 0);
                    } else {
                        const float x = S[u][0][r];
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), rc, off, 0, 0);
                    }
                }
        }

        phase();
        const int lane2 = (int)fresh((uint32_t)tid) & 63, li = lane2 & 15, grp = lane2 >> 4;
        // the fold
        if constexpr (fold.value) {
            // one column tile after the other: K^T is read once for each, and
            // V w of one tile only is held (both would spill the prefetch)
            const float gamma = sm.eG[b][CH - 1];
            #pragma unroll
            for (int t = 0; t < NT; ++t) {
                bf16x8 wh[2], wlo[2];
                #pragma unroll
                for (int mm = 0; mm < 2; ++mm) {
                    phase();
                    if constexpr (F32) {
                        wh[mm] = trn(sm.vw[0], VP, 32 * mm, 16 * NT * wave + 16 * t, li, grp);
                        wlo[mm] = trn(sm.vw[F32 ? 1 : 0], VP, 32 * mm, 16 * NT * wave + 16 * t, li, grp);
                    } else {
                        const f32x4 w0 = *reinterpret_cast<const f32x4*>(&sm.w[b][32 * mm + 8 * grp]);
                        const f32x4 w1 = *reinterpret_cast<const f32x4*>(&sm.w[b][32 * mm + 8 * grp + 4]);
                        weigh(trn(sm.v[0], VP, 32 * mm, 16 * NT * wave + 16 * t, li, grp), w0, w1, wh[mm], wlo[mm]);
                    }
                }
                #pragma unroll
                for (int u = 0; u < NU; ++u) {
                    if (u % 2 == 0) phase();
                    f32x4 D = {0.f, 0.f, 0.f, 0.f};
                    #pragma unroll
                    for (int mm = 0; mm < 2; ++mm) {
                        const bf16x8 kh = trk(sm.k[0], KP, 32 * mm, u, li, grp);
                        D = mma(kh, wh[mm], D);
                        D = mma(kh, wlo[mm], D);
                        if (F32) D = mma(trk(sm.k[NL - 1], KP, 32 * mm, u, li, grp), wh[mm], D);
                    }
                    #pragma unroll
                    for (int r = 0; r < 4; ++r) S[u][t][r] = __builtin_fmaf(gamma, S[u][t][r], D[r]);
                }
            }
        }
        // V operands of P V: V is overwritten after the barrier
        phase();
        bf16x8 vo[2][NT], vl[2][NT];
        #pragma unroll
        for (int mm = 0; mm < 2; ++mm)
            #pragma unroll
            for (int t = 0; t < NT; ++t) {
                vo[mm][t] = tra(sm.v[0], VP, 32 * mm, 16 * NT * wave + 16 * t, li, grp);
                if (F32) vl[mm][t] = tra(sm.v[NL - 1], VP, 32 * mm, 16 * NT * wave + 16 * t, li, grp);
            }
        lds_barrier();

        // o = scale (exp(G) X + P V)
        const rsrc_t ro = make_rsrc_u32(reinterpret_cast<const char*>(p.o) + c * CH * o_row,
                                        chunk_rows(p.T, c) * (uint32_t)o_row);
        const uint32_t oo = fresh(ooff);
        #pragma unroll
        for (int rb = 0; rb < 4; ++rb) {
            if (rb > 0) phase();
            f32x4 po[NT];
            #pragma unroll
            for (int t = 0; t < NT; ++t) po[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            #pragma unroll
            for (int pr = 0; pr <= rb / 2; ++pr) {
                const int unit = rb < 2 ? rb : 2 * rb - 2 + pr;
                const bf16x8 ph = *reinterpret_cast<const bf16x8*>(&sm.p[unit][0][8 * lane]);
                const bf16x8 pl = *reinterpret_cast<const bf16x8*>(&sm.p[unit][1][8 * lane]);
                #pragma unroll
                for (int t = 0; t < NT; ++t) {
                    po[t] = mma(ph, vo[pr][t], po[t]);
                    po[t] = mma(pl, vo[pr][t], po[t]);
                    if (F32) po[t] = mma(ph, vl[pr][t], po[t]);
                }
            }
            const f32x4 eg = *reinterpret_cast<const f32x4*>(&sm.eG[b][16 * rb + 4 * grp]);
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t off = oo + (uint32_t)(16 * rb + r) * (uint32_t)o_row;
                if constexpr (NT == 2) {
                    const f32x2 x = {p.scale * __builtin_fmaf(eg[r], acc[0][rb][r], po[0][r]),
                                     p.scale * __builtin_fmaf(eg[r], acc[NT - 1][rb][r], po[NT - 1][r])};
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), ro, off, 0, 0);
                } else {
                    const float x = p.scale * __builtin_fmaf(eg[r], acc[0][rb][r], po[0][r]);
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), ro, off, 0, 0);
                }
            }
        }
    };

    phase();
    load_g(c0);
    load(c0);
    tables((int)(c0 & 1));
    load_g(c0 + 1);
    lds_barrier();
    // the state after the segment's last chunk is the next segment's, which
    // the first launch has already formed; only the final state is wanted
    const int64_t cf = last_seg && p.final_state ? c1 : c1 - 1;
    #pragma unroll 1
    for (int64_t c = c0; c < cf; ++c) chunk(c, std::true_type{});
    if (c0 <= cf && cf < c1) chunk(cf, std::false_type{});

    if (last_seg && p.final_state && jok) {
        #pragma unroll
        for (int u = 0; u < NU; ++u)
            #pragma unroll
            for (int r = 0; r < 4; ++r) {
                float* a = p.final_state + ((int64_t)h * DK + 32 * (u >> 1) + 8 * grp + 4 * (u & 1) + r) * dv + jl;
                if constexpr (NT == 2) *reinterpret_cast<f32x2*>(a) = f32x2{S[u][0][r], S[u][NT - 1][r]};
                else *a = S[u][0][r];
            }
    }
}

template <int DK, bool F32, int NT>
hipError_t launch_seg(const SegParams& sp, hipStream_t stream) {
    const ScanParams& p = sp.s;
    const unsigned grid = (unsigned)((int64_t)sp.nseg * p.H * ((p.dv + 64 * NT - 1) / (64 * NT)));
    const void* fn = p.chunk_states ? reinterpret_cast<const void*>(&linattn_seg_kernel<DK, F32, NT, true>)
                                    : reinterpret_cast<const void*>(&linattn_seg_kernel<DK, F32, NT, false>);
    return launch_kernel(fn, dim3(grid), dim3(256), sp, stream);
}

template <int DK, int DA, bool F32>
hipError_t launch_fold(SegParams sp, hipStream_t stream) {
    const int per = (DK / DA) * (sp.s.dv / 16);
    sp.s.by_xcd = heads_by_xcd(sp.s.H, per);
    return launch_kernel(reinterpret_cast<const void*>(&linattn_fold_kernel<DK, DA, F32>),
                         dim3(head_slice_grid(sp.s.H, per)), dim3(64 * kFoldWaves), sp, stream);
}

template <int DK, bool F32>
hipError_t launch_t(const ScanParams& p, hipStream_t stream) {
    SegParams sp;
    sp.s = p;
    const SegPlan plan = linattn_seg_plan(p);
    sp.G = (int32_t)plan.G;
    sp.nseg = (int32_t)plan.nseg;
    if (sp.nseg == 1 && p.chunk_states) return hipErrorInvalidValue;  // (no such call: linattn_in_segments)
    if (sp.nseg > 1) {
        // Row blocks of 64 give twice the workgroups; whole heads of 128 rows
        // halve the reads of V and of the gates once the chip is full anyway
        // (the call, 16384 x 32: 252 us, with 64 rows 327; x 24: 214 and 296; at 16
        // heads 174 and 166, 2048 x 16 32.5 and 30.7).
        const hipError_t e = DK == 128 && p.H * (p.dv / 16) > 128 ? launch_fold<DK, DK, F32>(sp, stream)
                                                                  : launch_fold<DK, 64, F32>(sp, stream);
        if (e != hipSuccess) return e;
    }
    if constexpr (!F32)
        if (plan.cols == 128) return launch_seg<DK, F32, 2>(sp, stream);
    return launch_seg<DK, F32, 1>(sp, stream);
}

}  // namespace

hipError_t launch_linattn_seg(const ScanParams& p, hipStream_t stream) {
    // fp32 inputs keep hi and lo planes of K, Q and V in LDS; the scan
    // supports them at dk = 64.
    if (p.dk == 128 && !p.in_f32) return launch_t<128, false>(p, stream);
    if (p.dk == 64) return p.in_f32 ? launch_t<64, true>(p, stream) : launch_t<64, false>(p, stream);
    return hipErrorInvalidValue;
}

}  // namespace cap
