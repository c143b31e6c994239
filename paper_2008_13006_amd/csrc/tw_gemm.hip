// tw_gemm: C = A . (B * mask) for a packed tile-wise weight, one persistent kernel on gfx950.
//
// Paper: Sec. VI.  The kernel in Listing 1 loads A tiles while skipping pruned K positions with a
// per-tile mask vector, multiplies them with pre-processed B tiles on the matrix unit and stores C
// skipping pruned columns; equal-width tiles are batched to share A and batches run concurrently
// to even out the load.  The paper stores A transposed in global memory so that skipping a K
// position skips a whole row.  This kernel keeps those ideas and changes the mechanics for CDNA4:
//   * A stays row-major in HBM.  A workgroup loads a block of A rows ONCE with coalesced 16-byte
//     loads and writes it K-MAJOR into LDS (the transposition happens on chip).  Every tile the
//     workgroup works on then gathers its kept K rows from that copy with transposing LDS reads
//     (ds_read_b64_tr_b16) whose row addresses come from the tile's kept-K list: two reads
//     deliver the eight contraction values of an MFMA operand.  Skipping never touches global
//     memory and A is shared by many tiles (the role of batching).
//   * The compacted tile values are stored offline in MFMA operand order and go from global
//     memory (L2-resident) straight to registers, a few steps ahead of their use.
//   * Workgroups are persistent: one (row block, tile set) item each, further ones from an atomic
//     counter; inside a workgroup the waves pull tiles in the packer's dispatch order (the role of
//     stream concurrency).  When K does not fit in LDS, A is streamed through two LDS buffers.
//   * Pruned columns inside a tile's span are written as zeros together with the kept ones, as whole
//     128-byte lines of C, through a small per-wave LDS staging area.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "../../include/tw.h"
#include "tw_device.hpp"
#include "tw_format.h"

namespace {

constexpr int kWaves = TW_WAVES_PER_WG;
constexpr int kThreads = kWaves * 64;
// staging of A: resident K packs row pairs into 4-byte LDS writes, streamed K writes 2-byte values (see ATask)
constexpr bool kPairResident = true, kPairStream = false;
// B-operand steps in flight per wave: three; six for narrow tiles (at most two column blocks), whose steps
// are too short for three to cover the latency of an L2 hit and whose registers allow it
template <int NCB>
constexpr int prefetch_depth() { return NCB <= 2 ? 6 : 3; }
constexpr int kIdxAhead = 6;  // steps the K indices are requested ahead (they feed the LDS gather, which itself
                              // runs one step ahead of the MFMAs)

typedef short tw_i16x4 __attribute__((ext_vector_type(4)));
typedef float tw_f32x4 __attribute__((ext_vector_type(4)));

struct TwGemmParams {
    const unsigned char* blob;  // device copy
    const unsigned short* A;
    unsigned short* C;
    int* counters;              // [0] next item, [1] finished workgroups
    const unsigned short* bias; // fused epilogue: N values of the storage type, or null
    int act;                    // fused epilogue: tw_act
    long lda, ldc;
    int M, K, N, T;
    int k_chunk, n_chunks, G;
    int n_mblocks, n_seg, n_items;
    int tiles_per_set;          // MODE 2: tiles a workgroup holds (1..4: that many of the multiplying waves have one)
    int row_step;               // rows (tokens) from one row block to the next: 32*MS, or fewer (row-major boundary) so
                                // that the row blocks fill the last round of workgroups; rows past it are not stored
    unsigned at_pitch;          // bytes between K rows of the LDS copy of A (32*MS rows of A wide, padded)
    unsigned abuf_bytes;        // size of one LDS copy of A (streamed K uses two)
    unsigned stage_off;         // LDS offset of the per-wave staging areas
    unsigned misc_off;          // LDS offset of two ints (item, tile counter)
    uint64_t off_sched_desc, off_step_ptr, off_goff, off_dpos, off_bvals, off_zero_ptr, off_zero_cols, off_urow, off_ucnt;
    uint64_t off_ew_ptr, off_ew_goff, off_ew_b, off_xm_ptr, off_xm_goff, off_xm_b, off_zero_xc;
    int has_ew;                 // the blob carries an element-wise residual (TEW)
    uint64_t off_xc_tile_ptr, off_xc_col, off_xc_ptr, off_xc_k, off_xc_v;
    unsigned xbuf_off;          // LDS offset of the per-wave areas for residual-only columns (TEW), 0: the tiles' kernel
                                // leaves those columns to the pass of their own
    int stream_stores;          // rows of the output start on 128-byte boundaries: stores that complete whole lines
                                // may carry the streaming hint
    unsigned urow_off;          // LDS offset of the loading waves' row lists (transposed, streamed K, few tiles), 0: none
    // split K (streamed K, wave per tile, few row blocks): the K chunks are cut into n_parts runs of chunks_per_part
    // and an item is (part, tile set, row block); the tiles' fp32 results go to `partials`
    // ([part][row block][tile in dispatch order][MS][NCB][4 register groups][64 lanes][4]) and
    // tw_splitk_reduce_kernel adds them up in the order of the parts and stores C.  n_parts = 1: no split.
    int n_parts, chunks_per_part;
    float* partials;
    int team_shift;             // tw_team_kernel: log2 of the waves that share a tile (8, 4 or 2)
    int rows_group;             // tw_rows_kernel: token blocks that are walked together (see there)
};

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
// bytes between K rows of the LDS copy of A: 32*MS rows of A wide, padded by 8 (a compile-time value, so that the
// eight K rows a staging request writes to are immediate offsets of its LDS writes, not a multiplication each)
template <int MS> constexpr unsigned at_pitch_of() { return 64u * MS + 8u; }
// one past the last row of the row block that starts at row0
__device__ __forceinline__ int block_end(const TwGemmParams& p, int row0) {
    const int e = row0 + p.row_step;
    return e < p.M ? e : p.M;
}
// Returns x, but hides where it came from: values derived from the result are recomputed where they
// are used instead of being hoisted out of the persistent loop and kept (or spilled) across phases.
__device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Wave-uniform copy of a schedule descriptor, in SGPRs.  The packed weight is read-only for the
// kernel, so descriptors are read through the constant address space: the compiler then uses scalar
// loads, which cost no vector registers and whose wait (lgkmcnt) does not depend on the wave's
// outstanding vector stores.  The compiler places the wait at the first use, so a descriptor requested
// early arrives while other work runs.
struct TileU {
    int w, span_start, span_w, nsteps, tile, step_ptr, first_step, xc;
};
typedef const __attribute__((address_space(4))) int* tw_const_int_ptr;
__device__ __forceinline__ TileU fetch_tile(const TwGemmParams& p, int ti) {
    const uint64_t a = (uint64_t)(p.blob + p.off_sched_desc) + 32ull * (unsigned)ti;
    // the address is wave-uniform; say so to the compiler
    const uint64_t ua = ((uint64_t)(unsigned)uni((int)(a >> 32)) << 32) | (unsigned)uni((int)(unsigned)a);
    tw_const_int_ptr d = (tw_const_int_ptr)ua;
    TileU u;
    u.w = d[0]; u.span_start = d[1]; u.span_w = d[2]; u.nsteps = d[3];
    u.tile = d[4]; u.step_ptr = d[5]; u.first_step = d[6]; u.xc = d[7];
    return u;
}

// Element idx of a read-only int table, wave-uniform, through a scalar load (see fetch_tile).
__device__ __forceinline__ int fetch_int(const int* table, int idx) {
    const uint64_t a = (uint64_t)(table + idx);
    const uint64_t ua = ((uint64_t)(unsigned)uni((int)(a >> 32)) << 32) | (unsigned)uni((int)(unsigned)a);
    return *(tw_const_int_ptr)ua;
}

// Cooperative load of A[row0 .. row0+32*MS) x [k0, k0+kw) into LDS, transposed: LDS row k (pitch
// at_pitch bytes) holds the 32*MS values A[row0 .. , k0+k].  Row k_chunk of the LDS copy is kept zero
// for padded contraction slots; rows k_chunk+1 .. k_chunk+8 take the writes of absent pieces.
// A lane always reads 16-byte pieces (8 columns of one row).  Two ways of cutting the work into tasks:
//   PAIR = false (streamed K): a task is 8 rows x 64 columns; lane l reads piece l%8 of row l/8 (a wave
//     instruction reads 128 contiguous bytes of 8 rows, what streams best from HBM) and scatters its
//     values with eight 2-byte LDS writes.  One request per task.
//   PAIR = true (resident K): a task is 32 rows x 32 columns; lane l reads piece l/16 of the two rows
//     2*(l%16) and 2*(l%16)+1, and the two rows' values of a column go into one 32-bit word: eight
//     4-byte LDS writes per two requests, whose 64 lanes hit 64 different banks (the four pieces lie 16
//     banks apart, the 16 row pairs in consecutive words).  Two requests per task.
// Wave w takes tasks w, w+stride, ...  Neither the loads nor the LDS writes carry branches: a request
// for an absent piece re-reads a valid one and its values go to the spare rows, so all requests of a
// batch are outstanding together.  lda is a multiple of 8 elements, so the bytes past column K-1 of a
// row still belong to that row's pitch; they are dropped at the LDS write (only a width that is not a
// multiple of 8 needs that test).  BATCH counts requests.
template <int BATCH>
struct ARegs {
    tw_u32x4 v[BATCH];
};

// A 16-byte request for activations.  NTA (compile time, one kernel variant each): with the streaming hint when this
// workgroup is the only one that reads these rows (one set of tiles per row block: the rows then do not push the
// packed weights out of the L2; 2 to 6 us on the streamed workloads), plain when the tiles of a row block are split
// into sets whose workgroups read the same rows one after the other (the later ones then hit in the L2; the skewed
// FFN-down of BERT-large: 45 us against 49, transposed 41 against 50).
template <bool NTA>
__device__ __forceinline__ tw_u32x4 load_a16(const unsigned short* src) {
    if constexpr (NTA) return tw_load16_stream(src);
    else return *(const tw_u32x4*)src;
}

template <int MS, bool PAIR>
struct ATask {
    int row, oc;      // (first) row of the lane, 16-byte piece of the row
    bool have;
    __device__ __forceinline__ ATask(int t, int kw, int lane) {
        const int octets = (kw + 7) >> 3;           // 16-byte pieces per row
        if constexpr (PAIR) {
            const int tasks = MS * ((octets + 3) >> 2);
            const int tc = t < tasks ? t : tasks - 1;
            row = (tc % MS) * 32 + 2 * (lane & 15);
            const int o = (tc / MS) * 4 + (lane >> 4);
            have = t < tasks && o < octets;
            oc = o < octets ? o : octets - 1;
        } else {
            constexpr int RG = 4 * MS;              // groups of 8 rows
            const int tasks = RG * ((octets + 7) >> 3);
            const int tc = t < tasks ? t : tasks - 1;
            row = (tc % RG) * 8 + (lane >> 3);
            const int o = (tc / RG) * 8 + (lane & 7);
            have = t < tasks && o < octets;
            oc = o < octets ? o : octets - 1;
        }
    }
};
template <int MS, bool PAIR>
__device__ __forceinline__ int a_tasks(int kw) {
    const int octets = (kw + 7) >> 3;
    return PAIR ? MS * ((octets + 3) >> 2) : 4 * MS * ((octets + 7) >> 3);
}

// requests tasks t0, t0+stride, ... of the block (BATCH requests); stride = number of loading waves
template <int MS, int BATCH, bool PAIR, bool NTA = true>
__device__ __forceinline__ void a_issue(const TwGemmParams& p, ARegs<BATCH>& ar, int row0, int k0, int kw, int t0,
                                        int lane_in, int stride = kWaves) {
    const int lane = fresh(lane_in);
    const int mend = block_end(p, row0);
    if constexpr (PAIR) {
        static_assert(BATCH % 2 == 0, "two requests per task");
#pragma unroll
        for (int b = 0; b < BATCH / 2; ++b) {
            const ATask<MS, true> t(t0 + b * stride, kw, lane);
            int g0 = row0 + t.row, g1 = g0 + 1;
            g0 = g0 < mend ? g0 : mend - 1;           // rows past the block's end: any valid row, never stored
            g1 = g1 < mend ? g1 : mend - 1;
            // (plain loads: with K resident the streaming hint measured 1.5 us slower on the BERT-base shapes;
            // the streamed paths below gain 2 to 6 us from it)
            ar.v[2 * b] = *(const tw_u32x4*)(p.A + (long)g0 * p.lda + (k0 + t.oc * 8));
            ar.v[2 * b + 1] = *(const tw_u32x4*)(p.A + (long)g1 * p.lda + (k0 + t.oc * 8));
        }
    } else {
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const ATask<MS, false> t(t0 + b * stride, kw, lane);
            int grow = row0 + t.row;
            grow = grow < mend ? grow : mend - 1;
            ar.v[b] = load_a16<NTA>(p.A + (long)grow * p.lda + (k0 + t.oc * 8));
        }
    }
}

// writes what a_issue requested into the LDS copy `at`
template <int MS, int BATCH, bool PAIR>
__device__ __forceinline__ void a_commit(const TwGemmParams& p, const ARegs<BATCH>& ar, unsigned char* at, int kw, int t0,
                                         int lane_in, int stride = kWaves) {
    const int lane = fresh(lane_in);
    const int dump = p.k_chunk + 1;
    const bool tail = (kw & 7) != 0;                  // wave-uniform
    if constexpr (PAIR) {
#pragma unroll
        for (int b = 0; b < BATCH / 2; ++b) {
            const ATask<MS, true> t(t0 + b * stride, kw, lane);
            const int kcol = t.have ? t.oc * 8 : dump;
            unsigned char* dst = at + (unsigned)kcol * at_pitch_of<MS>() + t.row * 2;
            const unsigned x[4] = {ar.v[2 * b].x, ar.v[2 * b].y, ar.v[2 * b].z, ar.v[2 * b].w};
            const unsigned y[4] = {ar.v[2 * b + 1].x, ar.v[2 * b + 1].y, ar.v[2 * b + 1].z, ar.v[2 * b + 1].w};
            unsigned w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                w[i] = (i & 1) ? ((x[i >> 1] >> 16) | (y[i >> 1] & 0xFFFF0000u)) : ((x[i >> 1] & 0xFFFFu) | (y[i >> 1] << 16));
            if (!tail) {
#pragma unroll
                for (int i = 0; i < 8; ++i) *(unsigned*)(dst + (unsigned)i * at_pitch_of<MS>()) = w[i];
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (kcol + i < kw || kcol == dump) *(unsigned*)(dst + (unsigned)i * at_pitch_of<MS>()) = w[i];
            }
        }
    } else {
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
            const ATask<MS, false> t(t0 + b * stride, kw, lane);
            const int kcol = t.have ? t.oc * 8 : dump;
            unsigned char* dst = at + (unsigned)kcol * at_pitch_of<MS>() + t.row * 2;
            const unsigned w[4] = {ar.v[b].x, ar.v[b].y, ar.v[b].z, ar.v[b].w};
            if (!tail) {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    *(unsigned short*)(dst + (unsigned)i * at_pitch_of<MS>()) = (unsigned short)(w[i >> 1] >> (16 * (i & 1)));
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (kcol + i < kw || kcol == dump)
                        *(unsigned short*)(dst + (unsigned)i * at_pitch_of<MS>()) = (unsigned short)(w[i >> 1] >> (16 * (i & 1)));
            }
        }
    }
}

__device__ __forceinline__ void a_zero_row(const TwGemmParams& p, unsigned char* at, int bm, int tid) {
    if (tid < bm / 2) *(unsigned*)(at + (unsigned)p.k_chunk * p.at_pitch + tid * 4) = 0u;
}

// whole block, BATCH requests per wave in flight at a time (12 cover 64 rows x 768 columns)
template <int MS, int BATCH, bool PAIR, bool NTA = true>
__device__ __forceinline__ void load_a_block(const TwGemmParams& p, unsigned char* at, int row0, int k0, int kw,
                                             int wave, int lane, int tid) {
    const int tasks = a_tasks<MS, PAIR>(kw);
    for (int t0 = wave; t0 < tasks; t0 += kWaves * (PAIR ? BATCH / 2 : BATCH)) {
        ARegs<BATCH> ar;
        a_issue<MS, BATCH, PAIR, NTA>(p, ar, row0, k0, kw, t0, lane);
        a_commit<MS, BATCH, PAIR>(p, ar, at, kw, t0, lane);
    }
    a_zero_row(p, at, 32 * MS, tid);
}

// Operand registers of the main loop: packed B of the next kPrefetch steps, K indices of the next
// kIdxAhead steps.
template <int NCB>
struct StepRegs {
    tw_u16x8 bq[prefetch_depth<NCB>()][NCB];
    unsigned kk[kIdxAhead];
};

// Requests the packed B of step s (clamped to `last`) of a tile into slot `slot`.
template <int NCB, int STRIDE = NCB>
__device__ __forceinline__ void issue_b(StepRegs<NCB>& rg, int slot, const unsigned char* bl, int s, int last) {
    s = s < last ? s : last;
    const unsigned char* b = bl + ((long)s * STRIDE) * 1024;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        rg.bq[slot][cb] = *(const tw_u16x8*)(b + cb * 1024);
    }
}
// Requests this lane's two K indices of step s (clamped to `last`) into slot `slot`.
template <int NCB>
__device__ __forceinline__ void issue_k(StepRegs<NCB>& rg, int slot, const unsigned char* gk, int s, int last) {
    s = s < last ? s : last;
    rg.kk[slot] = *(const unsigned*)(gk + (long)s * 32);
}

// Requests the first steps of a tile; the range [s0, s1) must not be empty.  (STRIDE: column blocks of the tile, where the wave takes
// NCB of them.)
template <int NCB, int STRIDE = NCB>
__device__ __forceinline__ void prefetch_first_steps(StepRegs<NCB>& rg, const unsigned char* goff_tile,
                                                     const unsigned char* bvals_tile, int s0, int s1, int lane_in) {
    const int lane = fresh(lane_in);
    const unsigned char* gk = goff_tile + ((lane >> 5) * 4 + ((lane & 15) >> 2)) * 4;
    const unsigned char* bl = bvals_tile + lane * 16;
#pragma unroll
    for (int i = 0; i < kIdxAhead; ++i) issue_k<NCB>(rg, i, gk, s0 + i, s1 - 1);
#pragma unroll
    for (int i = 0; i < prefetch_depth<NCB>(); ++i) issue_b<NCB, STRIDE>(rg, i, bl, s0 + i, s1 - 1);
}

// Steps [s0, s1) (not empty) of one tile for this wave: gather A from LDS, stream packed B from global, MFMA.
// Expects the first steps in `rg` (prefetch_first_steps).  The packed B of step s+kPrefetch and the K
// indices of step s+kIdxAhead are requested while step s is multiplied, and the LDS gather of step s+1
// is issued before the MFMAs of step s, so both latencies hide behind MFMAs.  The loop body has no branches
// except its exits (requests past the last step are clamped to the last step and never used), which
// keeps the compiler's wait counts exact.
template <int DT, int MS, int NCB, int STRIDE = NCB>
__device__ __forceinline__ void run_steps(tw_f32x16 (&acc)[MS][NCB], StepRegs<NCB>& rg, const unsigned char* at,
                                          unsigned at_pitch, const unsigned char* goff_tile,
                                          const unsigned char* bvals_tile, int s0, int s1, int lane_in) {
    const int lane = fresh(lane_in);
    // lane l: 16-lane block b = l/16 covers rows 16*(b%2).. of the 32-row block, contraction half h = l/32;
    // inside the block, lane j addresses the K row of slot 8h + 4r + j/4 at row quad j%4
    const int h = lane >> 5, j = lane & 15;
    const unsigned lanebase = (unsigned)(((lane >> 4) & 1) * 16 + (j & 3) * 4) * 2;
    const unsigned char* gk = goff_tile + (h * 4 + (j >> 2)) * 4;   // this lane's two K indices of a step
    const unsigned char* bl = bvals_tile + lane * 16;
    const int last = s1 - 1;

    auto gather = [&](tw_u16x8 (&a)[MS], unsigned k2) {
        const unsigned a0 = (k2 & 0xFFFFu) * at_pitch + lanebase;
        const unsigned a1 = (k2 >> 16) * at_pitch + lanebase;
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) {
            const tw_i16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) tw_i16x4*)(at + a0 + ms * 64));
            const tw_i16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) tw_i16x4*)(at + a1 + ms * 64));
            a[ms] = tw_u16x8{(unsigned short)lo4[0], (unsigned short)lo4[1], (unsigned short)lo4[2],
                             (unsigned short)lo4[3], (unsigned short)hi4[0], (unsigned short)hi4[1],
                             (unsigned short)hi4[2], (unsigned short)hi4[3]};
        }
    };
    // two gather buffers used alternately (the unrolled body covers an even number of steps)
    // (both start defined: an undefined second buffer would be carried around the tile loop as a live value)
    tw_u16x8 a[2][MS];
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) a[1][ms] = tw_u16x8{0, 0, 0, 0, 0, 0, 0, 0};
    gather(a[0], rg.kk[0]);
    constexpr int kPrefetch = prefetch_depth<NCB>();
    constexpr int kUnroll = 6;                      // a multiple of 2, kPrefetch and kIdxAhead
    static_assert(kUnroll % 2 == 0 && kUnroll % kPrefetch == 0 && kUnroll % kIdxAhead == 0, "unroll factor");
    auto step = [&](int i, int s) {
        // the three stages keep this order: left alone, the instruction scheduler sinks the loads of
        // later steps next to their first use and the prefetch distance is lost
        gather(a[(i + 1) & 1], rg.kk[(i + 1) % kIdxAhead]);
        __builtin_amdgcn_sched_barrier(0);
        // the request for a column block of step s+kPrefetch follows the MFMAs that read its registers:
        // the requests reach the memory pipeline spread over the step instead of in a burst
        const int sb = (s + kPrefetch) < last ? (s + kPrefetch) : last;
        const unsigned char* bnext = bl + ((long)sb * STRIDE) * 1024;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
                acc[ms][cb] = tw_mfma<DT>(a[i & 1][ms], rg.bq[i % kPrefetch][cb], acc[ms][cb]);
            __builtin_amdgcn_sched_barrier(0);
            rg.bq[i % kPrefetch][cb] = *(const tw_u16x8*)(bnext + cb * 1024);
            __builtin_amdgcn_sched_barrier(0);
        }
        issue_k<NCB>(rg, i % kIdxAhead, gk, s + kIdxAhead, last);
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = s0;
    for (; s + kUnroll <= s1; s += kUnroll) {      // whole groups: no branch inside
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) step(i, s + i);
    }
    const int rest = s1 - s;                        // 0 .. kUnroll-1 steps left
#pragma unroll
    for (int i = 0; i < kUnroll - 1; ++i)
        if (i < rest) step(i, s + i);
}

// Epilogue of one tile for this wave.  In this kernel the activations are the FIRST MFMA operand, so a
// lane owns one packed column of the tile (n = lane % 32 of every 32-column block) and its registers
// are rows: register r of a 32 x 32 block is row 8*(r/4) + 4*(lane/32) + r%4, i.e. four consecutive
// rows per group of four registers.
//
// What the stores cost is the number of (128-byte line of C, store instruction) pairs, so every store
// instruction should cover whole lines.  The wave's LDS staging window therefore starts at the
// 64-column (128-byte) boundary at or below the tile's span and is up to four lines wide.  It is kept
// COLUMN-major: per destination column the four rows a lane holds are contiguous, so a lane stages
// the four rounded values of a register group with ONE 8-byte LDS write at the destination column of
// its packed column.  Two planes hold rows 0-3 and 4-7 of the eight rows of a pass (the two lane
// halves), each [256 columns][4 rows] followed by one spare slot per lane for absent columns; the
// second plane is skewed by 32 bytes so that reads of both planes use disjoint banks.  The window is
// cleared once per tile: every pass writes the same columns, so the pruned columns inside the span
// keep reading back as zeros.  The read-back uses the transposing LDS read (ds_read_b64_tr_b16):
// within 16 lanes, lane 4e+g supplies the address of column (c_g + e), rows (4 values), and lane
// 4g+x receives row x of columns c_g .. c_g+3.  Two such reads give a lane eight consecutive columns
// of one row (16 bytes), and a store instruction writes one 128-byte line of eight rows.  Groups that
// straddle the ends of the span go out as one 2-byte store per lane, end and pass.
// LDS instructions of one wave execute in order, so the wave needs no waits between its own writes
// and reads of the staging area, only compiler barriers; the writes of pass P+1 are issued behind
// the reads of pass P and ahead of the wait for them.
constexpr int kLineCols = 64;                       // columns in a 128-byte line of C
constexpr int kWinLines = 4;                        // lines per staging window
constexpr int kWinCols = kWinLines * kLineCols;     // 256
constexpr int kSpareOff = kWinCols * 8;             // spare slots behind the window of a plane
constexpr int kPlaneBytes = kWinCols * 8 + 32 * 8 + 32;
constexpr unsigned kStageBytes = 2 * kPlaneBytes;   // per wave
// Windows of kNarrowLines lines, where LDS has no room for more beside 64 rows of A (K from 921 to 1040).
// (32 rows of A stream the packed weights twice as often.  Before -> now: 4321 x 1000 -> 1234 (G = 32) 27.1 -> 22.5 us, 14528 x 1024 -> 2188
// (G = 32) 75 -> 50, 10752 x 960 -> 3328 with GELU 82 -> 60, 31710 x 1019 -> 1472 with GELU 106 -> 90.  A span wider than the window
// takes several, which costs the wave its staging again.)
constexpr int kNarrowLines = 2;
template <int WL> constexpr int plane_bytes() { return WL * kLineCols * 8 + 32 * 8 + 32; }
static_assert(plane_bytes<kWinLines>() == kPlaneBytes && plane_bytes<kNarrowLines>() % 16 == 0 && (plane_bytes<kNarrowLines>() / 4) % 16 == 8, "plane skew");
constexpr unsigned kNarrowStageBytes = 2 * plane_bytes<kNarrowLines>();
static_assert(kPlaneBytes % 16 == 0 && (kPlaneBytes / 4) % 16 == 8, "plane skew");

__device__ __forceinline__ void tw_compiler_fence() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ tw_i16x4 tw_lds_read_tr(const unsigned char* a) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) tw_i16x4*)a);
}

// dpos: destination columns of this lane's packed columns (one per 32-column block), counted from the
// 8-aligned column at or below the span start.
// Fused epilogue (p.bias and / or p.act): `eb` holds the bias of this lane's packed columns and of the
// four columns lane, lane+64, .. of the first staging window (see fetch_epi_bias).
template <int NCB>
struct EpiBias {
    float col[NCB];
    float fill[kWinLines];
};

// Bias of this lane's packed columns.
template <int DT, int NCB>
__device__ __forceinline__ void fetch_col_bias(const TwGemmParams& p, const TileU& d, const unsigned (&dpos)[NCB], float (&col)[NCB]) {
    const int origin = d.span_start & ~7;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        col[cb] = p.bias != nullptr && dpos[cb] != 0xFFFFFFFFu ? tw_to_f32<DT>(p.bias[origin + (int)dpos[cb]]) : 0.f;
}

// Reads what store_tile needs of the bias.
template <int DT, int NCB>
__device__ __forceinline__ void fetch_epi_bias(const TwGemmParams& p, const TileU& d, const unsigned (&dpos)[NCB],
                                               EpiBias<NCB>& eb, int lane) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) eb.col[cb] = 0.f;
#pragma unroll
    for (int l = 0; l < kWinLines; ++l) eb.fill[l] = 0.f;
    if (p.bias != nullptr) {                                // wave-uniform
        const int origin = d.span_start & ~7, E = d.span_start + d.span_w;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            if (dpos[cb] != 0xFFFFFFFFu) eb.col[cb] = tw_to_f32<DT>(p.bias[origin + (int)dpos[cb]]);
        if (d.span_w != d.w) {                              // pruned columns inside the span: they hold act(bias)
            const int W0 = d.span_start & ~(kLineCols - 1);
#pragma unroll
            for (int l = 0; l < kWinLines; ++l) {
                const int c = W0 + l * kLineCols + lane;
                if (c >= d.span_start && c < E) eb.fill[l] = tw_to_f32<DT>(p.bias[c]);
            }
        }
    }
}

// The fused epilogue's arithmetic, in place on the accumulators and kept apart from the store code, so that
// the plain path's code and registers stay as they are.
template <int MS, int NCB>
__device__ __forceinline__ void apply_bias_act(tw_f32x16 (&acc)[MS][NCB], const EpiBias<NCB>& eb, int act) {
    // The (wave-uniform) choice of the activation is taken once per 32 x 32 block, not once around three loops
    // over all accumulators: with one big three-way branch the register allocator moves accumulators out to
    // scratch memory on every path, the plain bias included.
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            if (act == TW_ACT_GELU) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ms][cb][r] = tw_gelu(acc[ms][cb][r] + eb.col[cb]);
            } else if (act == TW_ACT_RELU) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float x = acc[ms][cb][r] + eb.col[cb];
                    acc[ms][cb][r] = x > 0.f ? x : 0.f;
                }
            } else {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ms][cb][r] += eb.col[cb];
            }
        }
}

// The same for pieces of four results, in the waves that store a part of a tile only (teams of waves, second kernel of a
// split-K product): they have one or two of a tile's 4 to 8 units.  The activation is bound by the vector ALU: with
// GELU on the accumulators of all units 512 rows of 768 -> 2304 took 13.7 us, this way 11.0.
template <int NV>
__device__ __forceinline__ void apply_bias_act4(tw_f32x4 (&v)[NV], const float (&bias)[NV], int act) {
    if (act == TW_ACT_GELU) {                               // wave-uniform
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[i][e] = tw_gelu(v[i][e] + bias[i]);
    } else {
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = v[i][e] + bias[i];
                v[i][e] = act == TW_ACT_RELU && !(x > 0.f) ? 0.f : x;
            }
    }
}

// FUSED: the kernel variant with the fused epilogue (a bias and / or an activation); the plain variant
// carries none of its code.  PART: a wave that stores a part of the tile; bias and activation have been applied (pruned
// columns inside the span still take theirs here).
template <int DT, int MS, int NCB, bool FUSED, bool PART = false, int WL = kWinLines>
__device__ __forceinline__ void store_tile(const TwGemmParams& p, const TileU& d, tw_f32x16 (&acc)[MS][NCB],
                                           unsigned char* stage, const unsigned (&dpos)[NCB], int row0, int lane_in,
                                           unsigned short* xbuf = nullptr,
                                           const int* xcols = nullptr,
                                           int pass0 = 0, int pass1 = 4 * MS) {
    // (pass0, pass1: the passes to run, each eight rows of the block; everything by default.  The second kernel
    // of a split-K product gives a wave one pass of a tile.)
    constexpr int kCols = WL * kLineCols, kSpare = kCols * 8, kPlane = plane_bytes<WL>();
    const int lane = fresh(lane_in);
    constexpr bool fused = FUSED;
    // Residual-only columns of a TEW blob inside this tile's span (Sec. IV-A "Hybrid Pattern": weights restored in a
    // column that the tile-wise pattern pruned altogether).  With K resident the tile that owns the span has computed
    // them (xc_columns) into `xbuf` (16-bit, [column][row % 8][row / 8]); every pass puts its eight rows of them into the staging
    // window, where the pruned columns otherwise read back as zeros - so they leave with the tile's own stores.
    const int nx = xbuf != nullptr ? (int)((unsigned)d.xc >> 26) : 0;   // wave-uniform
    EpiBias<NCB> eb;
    if constexpr (FUSED) {
        fetch_epi_bias<DT, NCB>(p, d, dpos, eb, lane);
        if constexpr (!PART) apply_bias_act<MS, NCB>(acc, eb, p.act);
    }
    const int h = lane >> 5, n = lane & 31;
    const int blk = lane >> 4, j = lane & 15;
    // read-back, as the lane that supplies an address: column offset e, group g -> (piece, row quad)
    const int in_piece = 2 * blk + (j & 1), in_rq = (j >> 1) & 1, in_e = j >> 2;
    // read-back, as the lane that receives: group g = j / 4, row x = j % 4 of the quad
    const int piece = 2 * blk + ((j >> 2) & 1), orow = 4 * (j >> 3) + (j & 3);
    const int trow = lane >> 3, tg = lane & 7;              // element-wise stores: row, element of a group
    const int S = d.span_start, E = d.span_start + d.span_w;
    const int W0 = S & ~(kLineCols - 1);
    const unsigned shift = (unsigned)((S & ~7) - W0);       // dpos counts from S & ~7
    constexpr int NP = 4 * MS;
    const int rows_left = block_end(p, row0) - (row0 + orow);   // pass P stores this lane's row iff 8P < rows_left
    for (int win0 = W0; win0 < E; win0 += kCols) {       // one window unless the span is very wide
        const int left = E - win0;
        const int nl = left >= kCols ? WL : (left + kLineCols - 1) / kLineCols;
        unsigned char* wpos[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const unsigned rel = dpos[cb] + shift - (unsigned)(win0 - W0);   // wraps for columns left of the window
            wpos[cb] = stage + h * kPlane + (rel < (unsigned)kCols ? rel * 8u : (unsigned)(kSpare + n * 8));
        }
        const unsigned char* rpos = stage + in_rq * kPlane + (8 * in_piece + in_e) * 8;
        bool okl[WL], whole[WL];
#pragma unroll
        for (int l = 0; l < WL; ++l) {
            const int col = win0 + l * kLineCols + piece * 8;
            okl[l] = l < nl && col >= S && col + 8 <= E;
            // the span covers this line from end to end (wave-uniform): nobody else writes into it
            whole[l] = p.stream_stores != 0 && win0 + l * kLineCols >= S && win0 + (l + 1) * kLineCols <= E;
        }
        unsigned short* cptr = p.C + (long)(row0 + orow) * p.ldc + (win0 + piece * 8);
        // partial groups at the two ends of the span, if they lie in this window (window-relative index)
        int g_first = -1, g_last = -1;
        if ((S & 7) != 0 && win0 == W0) g_first = (S - win0) >> 3;
        if ((E & 7) != 0 && left <= kCols) g_last = (E - 1 - win0) >> 3;
        const int colF = win0 + g_first * 8 + tg, colL = win0 + g_last * 8 + tg;   // this lane's element
        const bool inF = g_first >= 0 && colF >= S && colF < E;
        const bool inL = g_last >= 0 && colL >= S && colL < E;
        const unsigned char* ragbase = stage + (trow >> 2) * kPlane + (trow & 3) * 2;
        const unsigned char* ragF = ragbase + ((g_first < 0 ? 0 : g_first) * 8 + tg) * 8;
        const unsigned char* ragL = ragbase + ((g_last < 0 ? 0 : g_last) * 8 + tg) * 8;
        unsigned short* rptr = p.C + (long)(row0 + trow) * p.ldc;
        const int rag_left = block_end(p, row0) - (row0 + trow);

        // residual-only columns: lane l handles column l / 8 (and l / 8 + 8) of the tile's list, row l % 8 of a pass
        unsigned char* xpos[TW_XC_INLINE / 8];
#pragma unroll
        for (int g = 0; g < TW_XC_INLINE / 8; ++g) {
            xpos[g] = nullptr;
            const int j = 8 * g + (lane >> 3);
            if (j < nx) {
                const unsigned rel = (unsigned)(xcols[g] - win0);
                if (rel < (unsigned)kCols) xpos[g] = stage + ((lane >> 2) & 1) * kPlane + rel * 8u + (lane & 3) * 2;
            }
        }
        tw_u32x4 xq[TW_XC_INLINE / 8];                       // this lane's row of its columns, all passes
#pragma unroll
        for (int g = 0; g < TW_XC_INLINE / 8; ++g) {
            xq[g] = tw_u32x4{0u, 0u, 0u, 0u};
            if (nx > 0) xq[g] = *(const tw_u32x4*)(xbuf + (8 * g + (lane >> 3)) * 64 + (lane & 7) * 8);
        }
        auto write_pass = [&](int P) {
            const int ms = P >> 2, q = P & 3;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                tw_u32x2 v;
                v.x = (unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 0]) | ((unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 1]) << 16);
                v.y = (unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 2]) | ((unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 3]) << 16);
                *(tw_u32x2*)wpos[cb] = v;
            }
            if (nx > 0) {                                    // wave-uniform
#pragma unroll
                for (int g = 0; g < TW_XC_INLINE / 8; ++g)
                    if (xpos[g] != nullptr)
                        *(unsigned short*)xpos[g] = (unsigned short)(xq[g][P >> 1] >> (16 * (P & 1)));
            }
        };

        // clear both planes once: the passes all write the same columns.  With a fused epilogue a pruned
        // column holds act(bias) in every row instead of zero.
        tw_compiler_fence();
        if (!fused || d.span_w == d.w) {
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
#pragma unroll
                for (int i = 0; i < kCols * 8 / 1024; ++i)
                    *(tw_u32x4*)(stage + pl * kPlane + i * 1024 + lane * 16) = tw_u32x4{0u, 0u, 0u, 0u};
        } else {
#pragma unroll
            for (int l = 0; l < WL; ++l) {
                const int c = win0 + l * kLineCols + lane;
                float b = eb.fill[l];
                if (win0 != W0) b = (p.bias != nullptr && c >= S && c < E) ? tw_to_f32<DT>(p.bias[c]) : 0.f;   // later windows: read here
                const unsigned hv = (c >= S && c < E) ? (unsigned)tw_cvt<DT>(tw_activate(b, p.act)) : 0u;
                const tw_u32x2 v{hv | (hv << 16), hv | (hv << 16)};
                *(tw_u32x2*)(stage + (l * kLineCols + lane) * 8) = v;
                *(tw_u32x2*)(stage + kPlane + (l * kLineCols + lane) * 8) = v;
            }
        }
        tw_compiler_fence();
#pragma unroll
        for (int P = 0; P < NP; ++P)
            if (P == pass0) write_pass(P);
        tw_compiler_fence();
#pragma unroll
        for (int P = 0; P < NP; ++P) {
            if (P < pass0 || P >= pass1) continue;               // wave-uniform
            tw_i16x4 lo[WL], hi[WL];
#pragma unroll
            for (int l = 0; l < WL; ++l) {
                lo[l] = tw_lds_read_tr(rpos + l * (kLineCols * 8));
                hi[l] = tw_lds_read_tr(rpos + l * (kLineCols * 8) + 32);
            }
            const unsigned short eF = *(const unsigned short*)ragF;
            const unsigned short eL = *(const unsigned short*)ragL;
            tw_compiler_fence();
            if (P + 1 < NP && P + 1 < pass1) write_pass(P + 1);
            tw_compiler_fence();
#pragma unroll
            for (int l = 0; l < WL; ++l) {
                if (okl[l] && 8 * P < rows_left) {
                    const tw_u32x2 a = __builtin_bit_cast(tw_u32x2, lo[l]), b = __builtin_bit_cast(tw_u32x2, hi[l]);
                    if (whole[l]) tw_store16_stream(cptr + (long)(8 * P) * p.ldc + l * kLineCols, tw_u32x4{a.x, a.y, b.x, b.y});
                    else *(tw_u32x4_a2*)tw_opaque(cptr + (long)(8 * P) * p.ldc + l * kLineCols) = tw_u32x4{a.x, a.y, b.x, b.y};
                }
            }
            if (g_first >= 0) {                              // wave-uniform
                if (inF && 8 * P < rag_left) rptr[(long)(8 * P) * p.ldc + colF] = eF;
            }
            if (g_last >= 0) {
                if (inL && 8 * P < rag_left) rptr[(long)(8 * P) * p.ldc + colL] = eL;
            }
            // At most a few of this wave's stores stay in flight: a long queue of stores in the CU's memory
            // pipeline holds up the loads of the waves that are multiplying (no load of this wave is pending here).
            asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        }
        tw_compiler_fence();
    }
}

// ---- Transposed boundary (TRANS): At is K x M, Ct is N x M (Sec. VI "Memory Accesses Coalescing") ----
// With the activations stored transposed, a K row of the workgroup's block is 128 contiguous bytes in
// global memory and goes to its LDS row as it is: the LDS copy needs no transposition, and skipping a
// pruned K position skips a row, which is what the paper changes the layout for.  A tile's results are
// rows of Ct (one per kept column), each a whole 128-byte line per block of 64 tokens: no line of
// the output is shared between tiles, and pruned columns are whole lines of zeros.

// Staging of At[k0 : k0+kw, m0 : m0 + 32*MS) into LDS (row k - k0 at (k - k0) * at_pitch), cut into tasks
// of 64 / (4*MS) rows: a wave instruction reads whole rows of the block (128 bytes with MS = 2).  Pieces
// past the row's pitch re-read the last piece inside it (they belong to tokens >= M, whose results
// are never stored).  One request per task; absent rows go to the spare rows.
template <int MS>
struct AtTask {
    int krow, pc;     // chunk-local K row, 16-byte piece of the block's row
    bool have;
    __device__ __forceinline__ AtTask(int t, int kw, int lane) {
        constexpr int PPR = 4 * MS, RPI = 64 / PPR;      // pieces per row, rows per instruction
        const int k = t * RPI + lane / PPR;
        have = k < kw;
        krow = have ? k : kw - 1;
        pc = lane % PPR;
    }
};
template <int MS>
__device__ __forceinline__ int at_tasks(int kw) { return (kw + 64 / (4 * MS) - 1) / (64 / (4 * MS)); }

template <int MS, int BATCH, bool NTA = true>
__device__ __forceinline__ void at_issue(const TwGemmParams& p, ARegs<BATCH>& ar, int m0, int k0, int kw, int t0,
                                         int lane_in, int stride = kWaves) {
    const int lane = fresh(lane_in);
    const int pmax = (int)((p.lda - m0) >> 3) - 1;
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        const AtTask<MS> t(t0 + b * stride, kw, lane);
        const int pc = t.pc < pmax ? t.pc : pmax;
        ar.v[b] = load_a16<NTA>(p.A + (long)(k0 + t.krow) * p.lda + (m0 + pc * 8));
    }
}

template <int MS, int BATCH>
__device__ __forceinline__ void at_commit(const TwGemmParams& p, const ARegs<BATCH>& ar, unsigned char* at, int kw, int t0,
                                          int lane_in, int stride = kWaves) {
    const int lane = fresh(lane_in);
    constexpr int PPR = 4 * MS;
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        const AtTask<MS> t(t0 + b * stride, kw, lane);
        const int krow = t.have ? t.krow : p.k_chunk + 1 + (lane / PPR) % 8;   // absent rows: the spare rows
        unsigned char* dst = at + (unsigned)krow * at_pitch_of<MS>() + t.pc * 16;
        *(tw_u32x2*)dst = tw_u32x2{ar.v[b].x, ar.v[b].y};
        *(tw_u32x2*)(dst + 8) = tw_u32x2{ar.v[b].z, ar.v[b].w};
    }
}

// The same with a row list: request b of the wave, row lane / 8 of it, stages chunk-local K row
// rows[8*b + lane/8] if that entry exists (entry number 8*(t0 + b*stride) + lane/8 below cnt).  K rows
// that no tile of the workgroup's set keeps are never read: with the activations transposed, skipping
// a K position skips a row of At (Sec. VI "Memory Accesses Coalescing").  `rows` is this wave's own
// copy in LDS of its entries of the chunk's list.
template <int BATCH>
__device__ __forceinline__ void at_issue_rows(const TwGemmParams& p, ARegs<BATCH>& ar, int m0, int k0,
                                              const unsigned short* rows, int cnt, int t0, int lane_in, int stride) {
    const int lane = fresh(lane_in);
    const int pmax = (int)((p.lda - m0) >> 3) - 1;
    const int pc = (lane & 7) < pmax ? (lane & 7) : pmax;
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        const int j = 8 * (t0 + b * stride) + (lane >> 3);
        const int krow = rows[8 * b + (lane >> 3)];
        ar.v[b] = tw_u32x4{0u, 0u, 0u, 0u};
        if (j < cnt) ar.v[b] = tw_load16_stream(p.A + (long)(k0 + krow) * p.lda + (m0 + pc * 8));
    }
}
template <int BATCH>
__device__ __forceinline__ void at_commit_rows(const TwGemmParams& p, const ARegs<BATCH>& ar, unsigned char* at,
                                               const unsigned short* rows, int cnt, int t0, int lane_in, int stride) {
    const int lane = fresh(lane_in);
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        const int j = 8 * (t0 + b * stride) + (lane >> 3);
        const int krow = j < cnt ? (int)rows[8 * b + (lane >> 3)] : p.k_chunk + 1 + (lane >> 3);
        unsigned char* dst = at + (unsigned)krow * at_pitch_of<2>() + (lane & 7) * 16;   // (64 tokens: MS = 2)
        *(tw_u32x2*)dst = tw_u32x2{ar.v[b].x, ar.v[b].y};
        *(tw_u32x2*)(dst + 8) = tw_u32x2{ar.v[b].z, ar.v[b].w};
    }
}

template <int MS, int BATCH, bool NTA = true>
__device__ __forceinline__ void load_at_block(const TwGemmParams& p, unsigned char* at, int m0, int k0, int kw, int wave,
                                              int lane, int tid) {
    const int tasks = at_tasks<MS>(kw);
    for (int t0 = wave; t0 < tasks; t0 += kWaves * BATCH) {
        ARegs<BATCH> ar;
        at_issue<MS, BATCH, NTA>(p, ar, m0, k0, kw, t0, lane);
        at_commit<MS, BATCH>(p, ar, at, kw, t0, lane);
    }
    a_zero_row(p, at, 32 * MS, tid);
}

// The two boundaries behind one name (TRANS: transposed).
// The common case of the streamed row-major staging written out (used where all eight waves stage): a chunk of
// 64 rows whose width is exactly what BATCH requests of STRIDE waves cover (8 * BATCH * STRIDE columns, 384 for
// 6 x 8), wave t0 < STRIDE.
// Same tasks and same LDS layout as a_issue / a_commit without row pairs (task t0 + b * STRIDE: rows
// 8 * (t % 8) .. + 7, columns 64 * (t / 8) .. + 63), but everything that does not depend on the lane is a
// constant here: one or two row pointers per chunk, one LDS address, immediate offsets (the general code
// spends about 75 instructions per request on its bookkeeping): 5 % on the FFN-down of BERT-base.
template <int BATCH, int STRIDE, bool NTA = true>
__device__ __forceinline__ void a_issue_full(const TwGemmParams& p, ARegs<BATCH>& ar, int row0, int k0, int t0, int lane_in) {
    static_assert(STRIDE == 4 || STRIDE == 8, "waves that share a chunk");
    const int lane = fresh(lane_in);
    const int mend = block_end(p, row0);
    constexpr int NRG = 8 / STRIDE;                       // row groups of this wave: t0, t0 + STRIDE, ..
    const unsigned short* rp[NRG];
#pragma unroll
    for (int g = 0; g < NRG; ++g) {
        int grow = row0 + (t0 + g * STRIDE) * 8 + (lane >> 3);
        grow = grow < mend ? grow : mend - 1;             // rows past the block's end: any valid row, never stored
        rp[g] = p.A + (long)grow * p.lda + (k0 + (lane & 7) * 8);
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b)
        ar.v[b] = load_a16<NTA>(rp[((b * STRIDE) & 7) / STRIDE] + ((b * STRIDE) >> 3) * 64);
}
template <int BATCH, int STRIDE>
__device__ __forceinline__ void a_commit_full(const ARegs<BATCH>& ar, unsigned char* at, int t0, int lane_in) {
    const int lane = fresh(lane_in);
    constexpr unsigned pitch = at_pitch_of<2>();
    unsigned char* base = at + (unsigned)((lane & 7) * 8) * pitch + (lane >> 3) * 2 + t0 * 16;
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
        unsigned char* dst = base + (unsigned)(((b * STRIDE) >> 3) * 64) * pitch + ((b * STRIDE) & 7) * 16;
        const unsigned w[4] = {ar.v[b].x, ar.v[b].y, ar.v[b].z, ar.v[b].w};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *(unsigned short*)(dst + (unsigned)i * pitch) = (unsigned short)(w[i >> 1] >> (16 * (i & 1)));
    }
}

template <int MS, int BATCH, bool TRANS, bool NTA = true>
__device__ __forceinline__ void stage_issue(const TwGemmParams& p, ARegs<BATCH>& ar, int r0, int k0, int kw, int t0, int lane,
                                            int stride = kWaves) {
    if constexpr (TRANS) {
        at_issue<MS, BATCH, NTA>(p, ar, r0, k0, kw, t0, lane, stride);
    } else {
        // (with four loading waves the written-out form measured no faster, 1.6 % slower on the conv workload)
        if (MS == 2 && stride == 8 && kw == 64 * BATCH) a_issue_full<BATCH, 8, NTA>(p, ar, r0, k0, t0, lane);
        else a_issue<MS, BATCH, kPairStream, NTA>(p, ar, r0, k0, kw, t0, lane, stride);
    }
}
template <int MS, int BATCH, bool TRANS>
__device__ __forceinline__ void stage_commit(const TwGemmParams& p, const ARegs<BATCH>& ar, unsigned char* at, int kw, int t0,
                                             int lane, int stride = kWaves) {
    if constexpr (TRANS) {
        at_commit<MS, BATCH>(p, ar, at, kw, t0, lane, stride);
    } else {
        if (MS == 2 && stride == 8 && kw == 64 * BATCH) a_commit_full<BATCH, 8>(ar, at, t0, lane);
        else a_commit<MS, BATCH, kPairStream>(p, ar, at, kw, t0, lane, stride);
    }
}

// Epilogue of one tile, transposed output.  Column block by column block, a lane (packed column n, its
// registers hold 4 consecutive tokens per group) writes its rounded values as 8-byte pieces into the
// wave's staging area [32 columns][32*MS tokens]; the rows are read back as 16-byte pieces and a store
// instruction writes whole rows of the block (128-byte lines with MS = 2) of 64 / (4*MS) rows of Ct.
// The destination row of a staged row comes from the lane that owns that packed column
// (ds_bpermute).  The pruned columns inside the tile's span are written as lines of zeros from the
// packer's list.
template <int DT, int MS, int NCB, bool FUSED, bool PART = false>
__device__ __forceinline__ void store_tile_t(const TwGemmParams& p, const TileU& d, tw_f32x16 (&acc)[MS][NCB],
                                             unsigned char* stage, const unsigned (&dpos)[NCB], int m0, int lane_in,
                                             int cb0 = 0, int cb1 = NCB, const unsigned short* xbuf = nullptr,
                                             bool zeros = true) {
    // (cb0, cb1: the column blocks to store, all by default; the lines of zeros go with column block 0.  The
    // second kernel of a split-K product gives a wave one column block of a tile.  zeros: whether this wave writes them.)
    constexpr int PPR = 4 * MS, RPI = 64 / PPR, PITCH = 64 * MS + 8;
    static_assert(32 * PITCH <= (int)kStageBytes, "transposed staging fits the wave's area");
    const int lane = fresh(lane_in);
    if constexpr (FUSED && !PART) {   // bias of this lane's packed columns (rows of Ct), activation in place
        EpiBias<NCB> eb;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            eb.col[cb] = (p.bias != nullptr && dpos[cb] != 0xFFFFFFFFu)
                             ? tw_to_f32<DT>(p.bias[(d.span_start & ~7) + (int)dpos[cb]]) : 0.f;
        apply_bias_act<MS, NCB>(acc, eb, p.act);
    }
    const int n = lane & 31, h = lane >> 5, rr = lane / PPR, pc = lane % PPR;
    const int origin = d.span_start & ~7;
    const int mleft = p.M - m0;                              // tokens of this block that exist
    const bool whole = 8 * pc + 8 <= mleft;                  // this lane's piece lies inside
    // a block of 64 tokens that exists in full is a whole 128-byte line of every row of Ct (wave-uniform)
    const bool stream = p.stream_stores != 0 && MS == 2 && mleft >= 64;
    auto put_piece = [&](long row, tw_u32x4 v) {
        unsigned short* dst = p.C + row * p.ldc + (m0 + 8 * pc);
        if (stream) {
            tw_store16_stream(dst, v);
        } else if (whole) {
            *(tw_u32x4*)tw_opaque(dst) = v;
        } else {
            const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (8 * pc + e < mleft) dst[e] = (unsigned short)(w[e >> 1] >> (16 * (e & 1)));
        }
    };
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        if (cb < cb0 || cb >= cb1) continue;                     // wave-uniform
        tw_compiler_fence();
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                tw_u32x2 v;
                v.x = (unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 0]) | ((unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 1]) << 16);
                v.y = (unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 2]) | ((unsigned)tw_cvt<DT>(acc[ms][cb][4 * q + 3]) << 16);
                *(tw_u32x2*)(stage + n * PITCH + (32 * ms + 8 * q + 4 * h) * 2) = v;
            }
        tw_compiler_fence();
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const int row = rr + RPI * i;                    // staged row = packed column 32*cb + row
            const tw_u32x2 lo = *(const tw_u32x2*)(stage + row * PITCH + pc * 16);
            const tw_u32x2 hi = *(const tw_u32x2*)(stage + row * PITCH + pc * 16 + 8);
            const unsigned dcol = (unsigned)__builtin_amdgcn_ds_bpermute(row * 4, (int)dpos[cb]);
            if (dcol != 0xFFFFFFFFu) put_piece((long)origin + (long)dcol, tw_u32x4{lo.x, lo.y, hi.x, hi.y});
        }
    }
    tw_compiler_fence();
    if (cb0 != 0 || !zeros) return;
    // lines of zeros for the pruned columns of the span
    const int* zp = (const int*)(p.blob + p.off_zero_ptr);
    const int* zc = (const int*)(p.blob + p.off_zero_cols);
    const int z0 = fetch_int(zp, d.tile), z1 = fetch_int(zp, d.tile + 1);
    // (`xbuf`: the rows of the span's residual-only columns that this tile has multiplied itself, [column][token])
    const signed char* zx = (const signed char*)(p.blob + p.off_zero_xc);
    for (int j = z0 + rr; j < z1; j += RPI) {
        const int col = zc[j];
        const int xs = xbuf != nullptr ? (int)zx[j] : -1;
        if (xs >= 0) {
            put_piece((long)col, *(const tw_u32x4*)(xbuf + xs * 64 + 8 * pc));
            continue;
        }
        unsigned v = 0u;
        if constexpr (FUSED) {   // a pruned column holds act(bias) for every token
            const unsigned hv = tw_cvt<DT>(tw_activate(p.bias != nullptr ? tw_to_f32<DT>(p.bias[col]) : 0.f, p.act));
            v = hv | (hv << 16);
        }
        put_piece((long)col, tw_u32x4{v, v, v, v});
    }
}

template <int MS, int NCB>
__device__ __forceinline__ void zero_acc(tw_f32x16 (&acc)[MS][NCB]) {
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[ms][cb][r] = 0.f;
}

// Element-wise residual of the TEW hybrid (Sec. IV-A): the weights kept outside the tile-wise pattern, in the
// tile's kept columns, are added to the tile's accumulators after the tile's own steps, by linearity.  The paper
// runs this part as a separate sparse product on the scalar cores; here it runs on the matrix cores out of the
// same LDS copy of A: per column block of 32 columns the packer lists the K rows in which the block has residual
// weights, 16 to a step, with the block's weights of those rows (mostly zeros).  One residual step is one such
// step of every column block: NCB gathers of A (each block has its own rows), NCB pieces of weights, MS * NCB
// MFMAs.  At 1 % of the weights a block of 32 columns touches about a quarter of the K rows, so the residual
// costs about as many MFMAs as the tile itself, where one fused multiply-add per row and weight on the vector
// units cost five times that.
// Same pipeline as run_steps: weights kDepth steps ahead, K rows kIdx steps ahead, the gather kRing - 1 column
// blocks ahead of the MFMAs that use it.
// Steps [s0, s1), not empty, of the tables `goff` (uint16 [steps][8][NCB][2]) and `bw` (16-bit [steps][NCB][64][8]).
template <int NCB>
struct BlockRegs {
    static constexpr int kDepth = 2, kIdx = NCB <= 2 ? 6 : 3;
    unsigned kk[kIdx][NCB];
    tw_u16x8 bq[kDepth][NCB];
};
template <int NCB>
__device__ __forceinline__ void block_load_k(BlockRegs<NCB>& r, int slot, const unsigned char* gk, int s, int last) {
    s = s < last ? s : last;
    const unsigned char* q = gk + (long)s * (32 * NCB);
    if constexpr (NCB == 4) {
        const tw_u32x4 t = *(const tw_u32x4*)q;
        r.kk[slot][0] = t.x; r.kk[slot][1] = t.y; r.kk[slot][2] = t.z; r.kk[slot][3] = t.w;
    } else if constexpr (NCB == 2) {
        const tw_u32x2 t = *(const tw_u32x2*)q;
        r.kk[slot][0] = t.x; r.kk[slot][1] = t.y;
    } else {
        r.kk[slot][0] = *(const unsigned*)q;
    }
}
// Requests the first steps of [s0, s1) (not empty).  The requests keep this order (first needed first): a wait for
// the first one must not wait for them all, and the loop's wait counts are the weaker of what its entry and its
// back edge allow.
template <int NCB>
__device__ __forceinline__ void request_block_steps(BlockRegs<NCB>& r, const unsigned char* goff, const unsigned char* bw,
                                                    int s0, int s1, int lane_in) {
    const int lane = fresh(lane_in);
    const unsigned char* gk = goff + ((lane >> 5) * 4 + ((lane & 15) >> 2)) * (NCB * 4);
    const unsigned char* bl = bw + lane * 16;
    const int last = s1 - 1;
#pragma unroll
    for (int i = 0; i < BlockRegs<NCB>::kIdx; ++i) {
        block_load_k<NCB>(r, i, gk, s0 + i, last);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < BlockRegs<NCB>::kDepth; ++i) {
        const int s = s0 + i < last ? s0 + i : last;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            r.bq[i][cb] = *(const tw_u16x8*)(bl + ((long)s * NCB + cb) * 1024);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}
// Expects the first steps in `r` (request_block_steps).
template <int DT, int MS, int NCB>
__device__ __forceinline__ void run_block_steps(tw_f32x16 (&acc)[MS][NCB], BlockRegs<NCB>& r, const unsigned char* at,
                                                unsigned at_pitch, const unsigned char* goff, const unsigned char* bw,
                                                int s0, int s1, int lane_in) {
    const int lane = fresh(lane_in);
    const int h = lane >> 5, j = lane & 15;
    const unsigned lanebase = (unsigned)(((lane >> 4) & 1) * 16 + (j & 3) * 4) * 2;
    const unsigned char* gk = goff + (h * 4 + (j >> 2)) * (NCB * 4);   // this lane's K rows of a step
    const unsigned char* bl = bw + lane * 16;
    const int last = s1 - 1;
    constexpr int kDepth = BlockRegs<NCB>::kDepth, kIdx = BlockRegs<NCB>::kIdx, kUnroll = 6;
    auto& kk = r.kk;
    auto& bq = r.bq;
    auto load_k = [&](int slot, int s) { block_load_k<NCB>(r, slot, gk, s, last); };
    auto gather = [&](tw_u16x8 (&a)[MS], unsigned k2) {
        const unsigned a0 = (k2 & 0xFFFFu) * at_pitch + lanebase;
        const unsigned a1 = (k2 >> 16) * at_pitch + lanebase;
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) {
            const tw_i16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) tw_i16x4*)(at + a0 + ms * 64));
            const tw_i16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) tw_i16x4*)(at + a1 + ms * 64));
            a[ms] = tw_u16x8{(unsigned short)lo4[0], (unsigned short)lo4[1], (unsigned short)lo4[2],
                             (unsigned short)lo4[3], (unsigned short)hi4[0], (unsigned short)hi4[1],
                             (unsigned short)hi4[2], (unsigned short)hi4[3]};
        }
    };
    constexpr int kRing = 2;   // (four buffers, the gather three column blocks ahead: no faster, 16 registers more)
    static_assert((kUnroll * NCB) % kRing == 0 && (kRing - 1 + NCB - 1) / NCB < kIdx, "ring of gather buffers");
    tw_u16x8 a[kRing][MS];
#pragma unroll
    for (int m = 0; m < kRing; ++m)
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) a[m][ms] = tw_u16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int m = 0; m < kRing - 1; ++m) gather(a[m], kk[m / NCB][m % NCB]);
    auto step = [&](int i, int s) {
        const int sb = (s + kDepth) < last ? (s + kDepth) : last;
        const unsigned char* bnext = bl + ((long)sb * NCB) * 1024;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            const int m = i * NCB + cb, ahead = cb + kRing - 1;
            gather(a[(m + kRing - 1) % kRing], kk[(i + ahead / NCB) % kIdx][ahead % NCB]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ms = 0; ms < MS; ++ms)
                acc[ms][cb] = tw_mfma<DT>(a[m % kRing][ms], bq[i % kDepth][cb], acc[ms][cb]);
            __builtin_amdgcn_sched_barrier(0);
            bq[i % kDepth][cb] = *(const tw_u16x8*)(bnext + cb * 1024);
            __builtin_amdgcn_sched_barrier(0);
        }
        load_k(i % kIdx, s + kIdx);
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = s0;
    for (; s + kUnroll <= s1; s += kUnroll) {
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) step(i, s + i);
    }
    const int rest = s1 - s;
#pragma unroll
    for (int i = 0; i < kUnroll - 1; ++i)
        if (i < rest) step(i, s + i);
}

template <int DT, int MS, int NCB>
__device__ __forceinline__ void add_ew_residual(const TwGemmParams& p, int tile, int chunk, tw_f32x16 (&acc)[MS][NCB],
                                                const unsigned char* at, unsigned at_pitch, int lane) {
    const int* ep = (const int*)(p.blob + p.off_ew_ptr);
    const int pi = tile * p.n_chunks + chunk;      // residual steps of this tile inside this K chunk (`at` holds the chunk)
    const int s0 = fetch_int(ep, pi), s1 = fetch_int(ep, pi + 1);
    if (s0 != s1) {
        BlockRegs<NCB> r;
        request_block_steps<NCB>(r, p.blob + p.off_ew_goff, p.blob + p.off_ew_b, s0, s1, lane);
        run_block_steps<DT, MS, NCB>(acc, r, at, at_pitch, p.blob + p.off_ew_goff, p.blob + p.off_ew_b, s0, s1, lane);
    }
}

// Residual-only columns inside a tile's span (weights restored in a column that the tile-wise pattern pruned
// altogether), row-major boundary: the first TW_XC_INLINE of a tile are multiplied like one more column block
// (packed column j = the tile's j-th such column; per K chunk the steps hold the K rows in which any of them has a
// weight) and put into `xbuf` (16-bit, [column][row % 8][row / 8]: the eight rows that one lane of the epilogue
// puts into the staging window, one per pass, lie side by side; act(. + bias) applied if FUSED), from where the
// tile's epilogue takes them.  With K streamed their fp32 sums wait between the chunks in the wave's staging
// area, which only the epilogue uses otherwise.
struct XcSteps {
    int s0, s1;
    BlockRegs<1> r;
};
__device__ __forceinline__ int xc_count(const TileU& d) { return (int)((unsigned)d.xc >> 26); }
// original column of the tile's residual-only columns l / 8 and l / 8 + 8 for lane l (what the epilogue needs)
__device__ __forceinline__ void xc_column_numbers(const TwGemmParams& p, const TileU& d, int (&col)[TW_XC_INLINE / 8], int lane) {
    const int x0 = d.xc & 0x3FFFFFF, nx = xc_count(d);
    const int* xcol = (const int*)(p.blob + p.off_xc_col);
#pragma unroll
    for (int g = 0; g < TW_XC_INLINE / 8; ++g) {
        col[g] = 0;
        const int j = 8 * g + (fresh(lane) >> 3);
        if (nx > 0) col[g] = xcol[x0 + (j < nx ? j : nx - 1)];   // wave-uniform condition
    }
}
__device__ __forceinline__ void xc_request(const TwGemmParams& p, const TileU& d, int chunk, XcSteps& x, int lane) {
    x.s0 = x.s1 = 0;
    if (xc_count(d) == 0) return;                            // wave-uniform
    const int* xp = (const int*)(p.blob + p.off_xm_ptr) + d.tile * p.n_chunks + chunk;
    x.s0 = fetch_int(xp, 0);
    x.s1 = fetch_int(xp, 1);
    if (x.s0 != x.s1) request_block_steps<1>(x.r, p.blob + p.off_xm_goff, p.blob + p.off_xm_b, x.s0, x.s1, lane);
}
template <int DT, int MS, bool FUSED>
__device__ __forceinline__ void xc_store(const TwGemmParams& p, const TileU& d, const tw_f32x16 (&acc)[MS][1],
                                         unsigned short* xbuf, int lane) {
    const int n = lane & 31, h = lane >> 5;
    if (n < xc_count(d)) {
        float bias = 0.f;
        if constexpr (FUSED)
            if (p.bias != nullptr) bias = tw_to_f32<DT>(p.bias[((const int*)(p.blob + p.off_xc_col))[(d.xc & 0x3FFFFFF) + n]]);
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int i = 0; i < 4; ++i) {                    // rows 32*ms + 8*q + 4*h + i, q = 0..3
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    v[q] = acc[ms][0][4 * q + i];
                    if constexpr (FUSED) v[q] = tw_activate(v[q] + bias, p.act);
                }
                tw_u32x2 o;
                o.x = (unsigned)tw_cvt<DT>(v[0]) | ((unsigned)tw_cvt<DT>(v[1]) << 16);
                o.y = (unsigned)tw_cvt<DT>(v[2]) | ((unsigned)tw_cvt<DT>(v[3]) << 16);
                *(tw_u32x2*)(xbuf + n * 64 + (4 * h + i) * 8 + 4 * ms) = o;
            }
    }
}
// Transposed boundary: a column is a row of Ct, `xbuf` is [column][token] and the epilogue writes its rows in place
// of the lines of zeros.
template <int DT, int MS, bool FUSED>
__device__ __forceinline__ void xc_store_t(const TwGemmParams& p, const TileU& d, const tw_f32x16 (&acc)[MS][1],
                                           unsigned short* xbuf, int lane) {
    const int n = lane & 31, h = lane >> 5;
    if (n < xc_count(d)) {
        float bias = 0.f;
        if constexpr (FUSED)
            if (p.bias != nullptr) bias = tw_to_f32<DT>(p.bias[((const int*)(p.blob + p.off_xc_col))[(d.xc & 0x3FFFFFF) + n]]);
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int q = 0; q < 4; ++q) {                    // tokens 32*ms + 8*q + 4*h .. + 3
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = acc[ms][0][4 * q + i];
                    if constexpr (FUSED) v[i] = tw_activate(v[i] + bias, p.act);
                }
                tw_u32x2 o;
                o.x = (unsigned)tw_cvt<DT>(v[0]) | ((unsigned)tw_cvt<DT>(v[1]) << 16);
                o.y = (unsigned)tw_cvt<DT>(v[2]) | ((unsigned)tw_cvt<DT>(v[3]) << 16);
                *(tw_u32x2*)(xbuf + n * 64 + 32 * ms + 8 * q + 4 * h) = o;
            }
    }
}
// K resident: everything at once
template <int DT, int MS, bool FUSED, bool TRANS>
__device__ __forceinline__ void xc_columns(const TwGemmParams& p, const TileU& d, XcSteps& x, const unsigned char* at,
                                           unsigned at_pitch, unsigned short* xbuf, int lane) {
    if (xc_count(d) == 0) return;                            // wave-uniform
    tw_f32x16 acc[MS][1];
    zero_acc<MS, 1>(acc);
    if (x.s0 != x.s1)
        run_block_steps<DT, MS, 1>(acc, x.r, at, at_pitch, p.blob + p.off_xm_goff, p.blob + p.off_xm_b, x.s0, x.s1, lane);
    if constexpr (TRANS) xc_store_t<DT, MS, FUSED>(p, d, acc, xbuf, lane);
    else xc_store<DT, MS, FUSED>(p, d, acc, xbuf, lane);
}
// K streamed: the sums of the 16 columns between chunks, fp32, piece (ms, q) of lane (h, n < 16) at float offset
// (((4 * ms + q) * 32 + 16 * h + n) * 4 of `area` (4 KB with 64 rows)
static_assert(TW_XC_INLINE == 16 && 2 * 4 * 32 * 16 <= (int)kStageBytes, "partial sums of the residual-only columns fit the staging area");
template <int MS>
__device__ __forceinline__ void xc_zero_partial(const TileU& d, unsigned char* area, int lane) {
    if (xc_count(d) == 0) return;                            // wave-uniform
#pragma unroll
    for (int i = 0; i < MS * 2; ++i) *(tw_u32x4*)(area + (i * 64 + lane) * 16) = tw_u32x4{0u, 0u, 0u, 0u};
}
template <int MS>
__device__ __forceinline__ void xc_load_partial(tw_f32x16 (&acc)[MS][1], const unsigned char* area, int lane) {
    zero_acc<MS, 1>(acc);
    const int n = lane & 31, h = lane >> 5;
    if (n < 16) {
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const tw_f32x4 v = *(const tw_f32x4*)(area + (((4 * ms + q) * 32 + 16 * h + n) * 16));
                acc[ms][0][4 * q + 0] = v.x; acc[ms][0][4 * q + 1] = v.y; acc[ms][0][4 * q + 2] = v.z; acc[ms][0][4 * q + 3] = v.w;
            }
    }
}
template <int DT, int MS>
__device__ __forceinline__ void xc_chunk(const TwGemmParams& p, const TileU& d, int chunk, const unsigned char* at,
                                         unsigned at_pitch, unsigned char* area, int lane) {
    XcSteps x;
    xc_request(p, d, chunk, x, lane);
    if (x.s0 == x.s1) return;                                // wave-uniform
    tw_f32x16 acc[MS][1];
    xc_load_partial<MS>(acc, area, lane);
    run_block_steps<DT, MS, 1>(acc, x.r, at, at_pitch, p.blob + p.off_xm_goff, p.blob + p.off_xm_b, x.s0, x.s1, lane);
    const int n = lane & 31, h = lane >> 5;
    if (n < 16) {
#pragma unroll
        for (int ms = 0; ms < MS; ++ms)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(tw_f32x4*)(area + (((4 * ms + q) * 32 + 16 * h + n) * 16)) =
                    tw_f32x4{acc[ms][0][4 * q + 0], acc[ms][0][4 * q + 1], acc[ms][0][4 * q + 2], acc[ms][0][4 * q + 3]};
    }
}
template <int DT, int MS, bool FUSED, bool TRANS>
__device__ __forceinline__ void xc_finish(const TwGemmParams& p, const TileU& d, const unsigned char* area,
                                          unsigned short* xbuf, int lane) {
    if (xc_count(d) == 0) return;                            // wave-uniform
    tw_f32x16 acc[MS][1];
    xc_load_partial<MS>(acc, area, lane);
    if constexpr (TRANS) xc_store_t<DT, MS, FUSED>(p, d, acc, xbuf, lane);
    else xc_store<DT, MS, FUSED>(p, d, acc, xbuf, lane);
}

// MODE 0: the K extent of a row block of 32*MS rows is resident in LDS, waves pull whole tiles.
// MODE 1: K streamed through two LDS buffers, row block of 64 rows (MS = 2), wave w owns tile 8*set + w.
// MODE 2: K streamed, row block of 64 rows (MS = 2), sets of 1, 2 or 4 tiles: of waves 0-3 wave w owns tile
//         tiles_per_set*set + w and multiplies, waves 4-7 do nothing but bring A into LDS, so the two kinds of
//         work overlap instead of taking turns (a wave's loads retire in order: a wave that waits for its packed
//         B also waits for every request for A it made before).
//         (Six multiplying and two loading waves were tried for weights of five or six tiles: the two
//         loading waves cannot keep up with the transposing LDS writes of the row-major boundary, 9 % slower
//         than MODE 1 on the FFN-down of BERT-base, and no gain on the transposed boundary.)
//         Row-major it serves TEW blobs and pitches from 2^23 elements; tw_stream_kernel has the rest.
// MODE 3: split K (below).  Row-major likewise: tw_part_kernel has the rest.
// Split K: a wave's fp32 results of its part of the K chunks, as they lie in the registers: piece (ms, cb, q) of
// lane l (registers 4q .. 4q+3 of acc[ms][cb]) at float offset (((ms * NCB + cb) * 4 + q) * 64 + l) * 4, so that
// every instruction writes (reads) 1 KB of consecutive memory.  32 KB per tile and part with 128-column tiles.
template <int MS, int NCB>
__device__ __forceinline__ void dump_partial(float* dst, const tw_f32x16 (&acc)[MS][NCB], int lane) {
    // dst is wave-uniform: said to the compiler, the 32 stores share one vector offset (the lane's) on a scalar
    // base instead of holding a vector address for every 4 KB of the range
    const uint64_t a = (uint64_t)dst;
    unsigned char* base = (unsigned char*)(((uint64_t)(unsigned)uni((int)(a >> 32)) << 32) | (unsigned)uni((int)(unsigned)a));
    const unsigned voff = (unsigned)lane * 16u;
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(tw_f32x4*)(base + ((ms * NCB + cb) * 4 + q) * 1024 + voff) =
                    tw_f32x4{acc[ms][cb][4 * q], acc[ms][cb][4 * q + 1], acc[ms][cb][4 * q + 2], acc[ms][cb][4 * q + 3]};
}

// EW: the variant for TEW blobs.  The code of the element-wise residual costs the kernels without it 1 to 2.5 %
// (registers: the widest variants sit at the limit of 256), so blobs without a residual run kernels without it.
// WL: lines of the epilogue's staging windows.
template <int DT, int MS, int NCB, int MODE, bool FUSED, bool TRANS, bool NTA = true, bool EW = false, int WL = kWinLines>
__global__ __launch_bounds__(kThreads) void tw_gemm_kernel(const TwGemmParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const bool has_ew = EW && p.has_ew != 0;
    const unsigned xbuf_off = EW ? p.xbuf_off : 0u;
    constexpr int MSB = MS;                       // 32-row blocks in the workgroup's row block
    constexpr int BM = 32 * MSB;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    unsigned char* stage = smem + p.stage_off + wave * (2 * plane_bytes<WL>());
    volatile int* misc = (volatile int*)(smem + p.misc_off);
    const int* step_ptr = (const int*)(p.blob + p.off_step_ptr);

    // The loop over the workgroup's items.  ROLE 0: every wave does the same (MODE 0 and 1); with MODE 2
    // the multiplying waves (ROLE 1) and the loading waves (ROLE 2) run copies of their own, with the
    // same barriers, so that neither carries the other's registers.
    // The first item of a workgroup is its own index, later ones come from the atomic counter.
    auto run_items = [&](auto role_tag) {
    constexpr int ROLE = decltype(role_tag)::value;
    int my_next = (int)blockIdx.x;   // thread 0: the item of the coming turn
    // loading waves: the first chunks of the coming item, requested during this item's epilogue
    ARegs<12> pre0, pre1;
    bool preloaded = false;
    int lists_of = -1;               // loading waves: the set whose row lists are in LDS
    int par = 0;                     // MODE 2: chunk c of the item lives in LDS buffer (c + par) % 2 (see the ring below)
    for (int turn = 0;; ++turn) {
        if (tid == 0) {
            misc[0] = my_next;
            misc[1] = 0;
        }
        __syncthreads();
        const int item = misc[0];
        if (item >= p.n_items) break;
        // the item after this one is requested now, so that the atomic's latency passes during this item's
        // work; the counter is touched only when there are more items than workgroups
        if (tid == 0) my_next = p.n_items > (int)gridDim.x ? (int)gridDim.x + atomicAdd(&p.counters[0], 1) : p.n_items;

        if constexpr (MODE == 0) {
            // the whole K extent of the row block stays in LDS; waves pull tiles of this item's set
            // (TRANS: transposed boundary, the row block is a block of tokens)
            const int mb = item / p.n_seg, seg = item - mb * p.n_seg;
            const int row0 = mb * p.row_step;
            // first tile of this wave: its descriptor is requested before A is staged
            int i = 0;
            if (lane == 0) i = atomicAdd((int*)&misc[1], 1);
            int ti = seg + uni(i) * p.n_seg;
            TileU next = fetch_tile(p, ti < p.T ? ti : 0);
            if constexpr (TRANS) load_at_block<MS, 12>(p, smem, row0, 0, p.K, wave, lane, tid);
            else load_a_block<MS, 12, kPairResident>(p, smem, row0, 0, p.K, wave, lane, tid);
            __syncthreads();
            while (ti < p.T) {
                const TileU d = next;
                // claim the next tile now so that its descriptor arrives during this tile's work
                if (lane == 0) i = atomicAdd((int*)&misc[1], 1);
                ti = seg + uni(i) * p.n_seg;
                next = fetch_tile(p, ti < p.T ? ti : 0);

                // destination columns of this lane's packed columns, needed only in the epilogue: request them now
                unsigned dpos[NCB];
                {
                    const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB;
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) dpos[cb] = dp[cb];
                }
                // residual-only columns of the tile's span (TEW): multiplied first, while the tile's own first
                // operands are on their way (their requests come first, so the wait for them is the shorter one)
                unsigned short* xbuf = nullptr;
                XcSteps xs;
                int xcols[TW_XC_INLINE / 8];
                if (xbuf_off != 0) {
                    xbuf = (unsigned short*)(smem + xbuf_off) + wave * (TW_XC_INLINE * 64);
                    if constexpr (!TRANS) xc_column_numbers(p, d, xcols, lane);
                    xc_request(p, d, 0, xs, lane);
                }
                StepRegs<NCB> rg;
                prefetch_first_steps<NCB>(rg, p.blob + p.off_goff + (long)d.first_step * 32,
                                          p.blob + p.off_bvals + (long)d.first_step * NCB * 1024, 0, d.nsteps, lane);
                if (xbuf != nullptr) xc_columns<DT, MS, FUSED, TRANS>(p, d, xs, smem, at_pitch_of<MS>(), xbuf, lane);
                tw_f32x16 acc[MS][NCB];
                zero_acc<MS, NCB>(acc);
                run_steps<DT, MS, NCB>(acc, rg, smem, at_pitch_of<MS>(), p.blob + p.off_goff + (long)d.first_step * 32,
                                           p.blob + p.off_bvals + (long)d.first_step * NCB * 1024, 0, d.nsteps, lane);
                if (has_ew) add_ew_residual<DT, MS, NCB>(p, d.tile, 0, acc, smem, at_pitch_of<MS>(), lane);
                if constexpr (TRANS) store_tile_t<DT, MS, NCB, FUSED>(p, d, acc, stage, dpos, row0, lane, 0, NCB, xbuf);
                else store_tile<DT, MS, NCB, FUSED, false, WL>(p, d, acc, stage, dpos, row0, lane, xbuf, xcols);
            }
            __syncthreads();  // everyone is done with the LDS copy of A and with misc[]
        } else if constexpr (MODE == 2) {
            // K streamed, multiplying waves and loading waves.  Chunk c is multiplied out of buffer c % 2
            // while the loading waves write chunk c+1 into the other buffer and request chunk c+3;
            // one barrier per chunk.
            constexpr int NMUL = kWaves / 2, NLD = kWaves - NMUL;
            constexpr int PB = 12;   // requests per loading wave and chunk: 64 rows x 384 columns in 4 waves
            const int set = item / p.n_mblocks, mb = item - set * p.n_mblocks;
            const int row0 = mb * p.row_step;
            const bool loader = wave >= NMUL;
            const int ti = set * p.tiles_per_set + wave;
            const bool active = wave < p.tiles_per_set && ti < p.T;      // (tiles_per_set <= NMUL: never a loading wave)
            const TileU d = fetch_tile(p, active ? ti : 0);
            const int* sp = step_ptr + d.step_ptr;
            const unsigned char* gt = p.blob + p.off_goff + (long)d.first_step * 32;
            const unsigned char* bt = p.blob + p.off_bvals + (long)d.first_step * NCB * 1024;
            auto chunk_width = [&](int c) {
                const int k0 = c * p.k_chunk;
                return (p.K - k0) < p.k_chunk ? (p.K - k0) : p.k_chunk;
            };
            if (tid < BM / 2) {
                *(unsigned*)(smem + (unsigned)p.k_chunk * p.at_pitch + tid * 4) = 0u;
                *(unsigned*)(smem + p.abuf_bytes + (unsigned)p.k_chunk * p.at_pitch + tid * 4) = 0u;
            }
            if constexpr (ROLE == 2) {
                const int lw = wave - NMUL;
                static_assert(PB == 12, "size of the carried register sets");
                // Transposed boundary: this wave's entries of the set's row lists, all chunks, in its own
                // piece of LDS ([chunk][8 * PB] rows, then [chunk] counts); filled when the set changes.
                constexpr int kListEntries = 8 * PB;
                unsigned short* my_rows = (unsigned short*)(smem + p.urow_off) + (long)lw * p.n_chunks * (kListEntries + 2);
                int* my_cnt = (int*)(my_rows + (long)p.n_chunks * kListEntries);
                const bool use_rows = TRANS && p.urow_off != 0;
                auto load_lists = [&](int st) {
                    const unsigned short* g = (const unsigned short*)(p.blob + p.off_urow) + (long)st * p.n_chunks * p.k_chunk;
                    const int* gc = (const int*)(p.blob + p.off_ucnt) + (long)st * p.n_chunks;
                    for (int c = 0; c < p.n_chunks; ++c) {
                        for (int e = lane; e < kListEntries; e += 64)
                            my_rows[c * kListEntries + e] = g[(long)c * p.k_chunk + 8 * (lw + (e >> 3) * NLD) + (e & 7)];
                        if (lane == 0) my_cnt[c] = gc[c];
                    }
                };
                // Across items: the ring of chunks (chunk c in LDS buffer (c + par) % 2, waiting in register set c % 2)
                // runs on into the NEXT item of the workgroup when that item has the same set of tiles: ring positions
                // n_chunks, n_chunks + 1, .. are its chunks 0, 1, ..  They are requested during this item's last chunks
                // and its chunk 0 is written to LDS while the multiplying waves work on this item's last chunk (the
                // buffers alternate, so that buffer is free), which is the state that start_item would otherwise only
                // begin to build when this item's steps are over.  With an odd number of chunks the buffers (`par`) and
                // the register sets change roles from one item to the next.
                // (`cross`, `nrow0`: set after the item's first barrier, where thread 0 has said which item comes next.)
                const bool ring = p.n_chunks >= 3;
                bool cross = false;
                int nrow0 = 0;
                auto issue_or_zero = [&](ARegs<PB>& ar, int c, int r0) {
                    const bool into_next = c >= p.n_chunks && cross && c - p.n_chunks < p.n_chunks;
                    if (c < p.n_chunks || into_next) {
                        if (into_next) { c -= p.n_chunks; r0 = nrow0; }
                        if (use_rows)
                            at_issue_rows<PB>(p, ar, r0, c * p.k_chunk, my_rows + c * kListEntries, uni(my_cnt[c]), lw, lane, NLD);
                        else
                            stage_issue<MSB, PB, TRANS, NTA>(p, ar, r0, c * p.k_chunk, chunk_width(c), lw, lane, NLD);
                    } else {
#pragma unroll
                        for (int b = 0; b < PB; ++b) ar.v[b] = tw_u32x4{0u, 0u, 0u, 0u};   // defined on every path
                    }
                };
                auto commit = [&](const ARegs<PB>& ar, int c) {
                    const bool into_next = c >= p.n_chunks && cross && c - p.n_chunks < p.n_chunks;
                    if (c < p.n_chunks || into_next) {
                        unsigned char* buf = smem + ((c + par) & 1) * p.abuf_bytes;          // by ring position
                        if (into_next) c -= p.n_chunks;
                        if (use_rows)
                            at_commit_rows<PB>(p, ar, buf, my_rows + c * kListEntries, uni(my_cnt[c]), lw, lane, NLD);
                        else
                            stage_commit<MSB, PB, TRANS>(p, ar, buf, chunk_width(c), lw, lane, NLD);
                    }
                };
                // chunk j waits in register set j % 2; the loop is unrolled by two so that the sets are
                // addressed statically.  The start of an item (chunk 0 in LDS, chunks 1 and 2 requested) was
                // done at the end of the previous item where there was one.
                ARegs<PB>& ar0 = pre0;
                ARegs<PB>& ar1 = pre1;
                auto start_item = [&](int r0) {
                    issue_or_zero(ar0, 0, r0);
                    issue_or_zero(ar1, 1, r0);
                    commit(ar0, 0);
                    issue_or_zero(ar0, 2, r0);
                };
                if (!preloaded) {
                    if (use_rows && set != lists_of) { load_lists(set); lists_of = set; }
                    start_item(row0);
                }
                __syncthreads();
                if (ring) {
                    const int nxt = misc[2];
                    cross = nxt < p.n_items && nxt / p.n_mblocks == set;
                    nrow0 = (nxt % p.n_mblocks) * p.row_step;
                }
                for (int c = 0; c < p.n_chunks; c += 2) {
                    commit(ar1, c + 1);
                    issue_or_zero(ar1, c + 3, row0);
                    __syncthreads();
                    if (c + 1 < p.n_chunks) {
                        commit(ar0, c + 2);
                        issue_or_zero(ar0, c + 4, row0);
                    }
                    __syncthreads();
                }
                // the multiplying waves are through with both buffers; the next item's first chunks are brought in
                // while they store this item's tiles, unless the ring has done that already
                __syncthreads();
                const int nxt = misc[2];
                preloaded = nxt < p.n_items;
                par ^= p.n_chunks & 1;
                if (preloaded && cross) {
                    if (p.n_chunks & 1) {        // ring positions n+1 and n+2 are the next item's chunks 1 and 2: sets 1 and 0 there
#pragma unroll
                        for (int b = 0; b < PB; ++b) { const tw_u32x4 t = ar0.v[b]; ar0.v[b] = ar1.v[b]; ar1.v[b] = t; }
                    }
                } else if (preloaded) {
                    const int nset = nxt / p.n_mblocks;
                    if (use_rows && nset != lists_of) { load_lists(nset); lists_of = nset; }
                    start_item((nxt % p.n_mblocks) * p.row_step);
                }
            } else {
                unsigned dpos[NCB];
                {
                    const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB;
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) dpos[cb] = dp[cb];
                }
                tw_f32x16 acc[MS][NCB];
                zero_acc<MS, NCB>(acc);
                // residual-only columns of the tile's span (TEW): their sums wait in the staging area between chunks
                unsigned short* xbuf = nullptr;
                int xcols[TW_XC_INLINE / 8];
                if (xbuf_off != 0 && active) {
                    xbuf = (unsigned short*)(smem + xbuf_off) + wave * (TW_XC_INLINE * 64);
                    if constexpr (!TRANS) xc_column_numbers(p, d, xcols, lane);
                    xc_zero_partial<MS>(d, stage, lane);
                }
                // the first steps of a chunk are requested at the end of the previous chunk's steps, so
                // they arrive while the workgroup meets at the barrier
                StepRegs<NCB> rg;
                // first steps of the chunks: b0 = first step of chunk c, b1 of chunk c+1, b2 of chunk c+2, read one
                // chunk ahead with scalar loads so that no chunk waits for them
                int b0 = fetch_int(sp, 0), b1 = fetch_int(sp, 1), b2 = fetch_int(sp, p.n_chunks < 2 ? p.n_chunks : 2);
                auto prefetch_steps = [&](int c0, int c1) {
                    if (active && c0 < c1) {
                        prefetch_first_steps<NCB>(rg, gt, bt, c0, c1, lane);
                    } else {                               // defined on every path
#pragma unroll
                        for (int i = 0; i < kIdxAhead; ++i) rg.kk[i] = 0u;
#pragma unroll
                        for (int i = 0; i < prefetch_depth<NCB>(); ++i)
#pragma unroll
                            for (int cb = 0; cb < NCB; ++cb) rg.bq[i][cb] = tw_u16x8{0, 0, 0, 0, 0, 0, 0, 0};
                    }
                };
                auto steps_of = [&](int c) {
                    const unsigned char* buf = smem + ((c + par) & 1) * p.abuf_bytes;
                    if (active && b0 < b1)
                        run_steps<DT, MS, NCB>(acc, rg, buf, at_pitch_of<MS>(), gt, bt, b0, b1, lane);
                    if (has_ew && active) add_ew_residual<DT, MS, NCB>(p, d.tile, c, acc, buf, at_pitch_of<MS>(), lane);
                    if (xbuf != nullptr) xc_chunk<DT, MS>(p, d, c, buf, at_pitch_of<MS>(), stage, lane);
                    // on to chunk c+1
                    b0 = b1; b1 = b2;
                    b2 = fetch_int(sp, c + 3 < p.n_chunks ? c + 3 : p.n_chunks);
                    if (c + 1 < p.n_chunks) prefetch_steps(b0, b1); else prefetch_steps(0, 0);
                };
                prefetch_steps(b0, b1);
                if (tid == 0) misc[2] = my_next;   // the loading waves look one item ahead (requested at the top of this turn)
                __syncthreads();
                for (int c = 0; c < p.n_chunks; c += 2) {
                    steps_of(c);
                    __syncthreads();
                    if (c + 1 < p.n_chunks) steps_of(c + 1);
                    __syncthreads();
                }
                __syncthreads();
                par ^= p.n_chunks & 1;
                if (active) {
                    if (xbuf != nullptr) xc_finish<DT, MS, FUSED, TRANS>(p, d, stage, xbuf, lane);
                    if constexpr (TRANS) store_tile_t<DT, MS, NCB, FUSED>(p, d, acc, stage, dpos, row0, lane, 0, NCB, xbuf);
                    else store_tile<DT, MS, NCB, FUSED>(p, d, acc, stage, dpos, row0, lane, xbuf, xcols);
                }
            }
        } else {
            // K is streamed in chunks through two LDS buffers: the requests for chunk c+1 go out before
            // the steps of chunk c and are written to the other buffer after them, one barrier per chunk.
            // Split K (MODE 3, few row blocks): the item also names a part of the chunks, [c_first, c_first + n_loc),
            // and a set may have fewer than eight tiles (the other waves then only bring in A); the tiles' fp32
            // results go to the workspace and a second kernel adds the parts up.  A kernel variant of its own, so
            // that the unsplit kernel carries none of this.
            constexpr bool SPLIT = MODE == 3;
            const int sp_item = item / p.n_mblocks, mb = item - sp_item * p.n_mblocks;
            const int part = SPLIT ? sp_item / p.n_seg : 0, set = sp_item - part * p.n_seg;
            const int c_first = SPLIT ? part * p.chunks_per_part : 0;
            const int n_loc = !SPLIT ? p.n_chunks
                              : (p.n_chunks - c_first) < p.chunks_per_part ? (p.n_chunks - c_first) : p.chunks_per_part;
            const int row0 = mb * p.row_step;
            const int ti = set * (SPLIT ? p.tiles_per_set : kWaves) + wave;
            const bool active = (!SPLIT || wave < p.tiles_per_set) && ti < p.T;
            const TileU d = fetch_tile(p, active ? ti : 0);
            constexpr int AB = 6;    // requests per wave and chunk: 64 rows x 384 columns in 8 waves
            // (chunk j of the item is chunk c_first + j of K and lives in LDS buffer j % 2)
            auto chunk_width = [&](int j) {
                const int k0 = (c_first + j) * p.k_chunk;
                return (p.K - k0) < p.k_chunk ? (p.K - k0) : p.k_chunk;
            };
            auto issue_or_zero = [&](ARegs<AB>& ar, int j) {
                if (j < n_loc) {
                    stage_issue<MSB, AB, TRANS, NTA>(p, ar, row0, (c_first + j) * p.k_chunk, chunk_width(j), wave, lane);
                } else {
#pragma unroll
                    for (int b = 0; b < AB; ++b) ar.v[b] = tw_u32x4{0u, 0u, 0u, 0u};   // defined on every path
                }
            };
            auto commit = [&](const ARegs<AB>& ar, int j) {
                if (j < n_loc) stage_commit<MSB, AB, TRANS>(p, ar, smem + (j & 1) * p.abuf_bytes, chunk_width(j), wave, lane);
            };
            // Split K: the item's first chunk is requested before anything waits for the tile's descriptor (the
            // descriptor, the table of first steps and the first packed weights are three dependent round trips to
            // memory, and an item is only a few chunks long); written to LDS below, behind the first requests for
            // packed weights.  (Not in the unsplit kernel: the registers it takes there cost more than it gains.)
            ARegs<AB> first;
            if constexpr (SPLIT) {
                issue_or_zero(first, 0);
            } else {
                const int kw = chunk_width(0);
                if constexpr (TRANS) load_at_block<MSB, AB, NTA>(p, smem, row0, c_first * p.k_chunk, kw, wave, lane, tid);
                else load_a_block<MSB, AB, kPairStream, NTA>(p, smem, row0, c_first * p.k_chunk, kw, wave, lane, tid);
                a_zero_row(p, smem + p.abuf_bytes, BM, tid);
            }
            unsigned dpos[NCB];
            if constexpr (!SPLIT) {
                const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB;
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) dpos[cb] = dp[cb];
            }
            tw_f32x16 acc[MS][NCB];
            zero_acc<MS, NCB>(acc);
            // residual-only columns of the tile's span (TEW): their sums wait in the staging area between chunks
            // (a split-K plan leaves them to the pass of their own)
            unsigned short* xbuf = nullptr;
            int xcols[TW_XC_INLINE / 8];
            if constexpr (!SPLIT) {
                if (xbuf_off != 0 && active) {
                    xbuf = (unsigned short*)(smem + xbuf_off) + wave * (TW_XC_INLINE * 64);
                    if constexpr (!TRANS) xc_column_numbers(p, d, xcols, lane);
                    xc_zero_partial<MS>(d, stage, lane);
                }
            }
            const int* sp = step_ptr + d.step_ptr;
            const unsigned char* gt = p.blob + p.off_goff + (long)d.first_step * 32;
            const unsigned char* bt = p.blob + p.off_bvals + (long)d.first_step * NCB * 1024;
            // Requests run kAhead chunks ahead of the steps: two where the registers allow it (narrow
            // tiles), so that a chunk is always on its way from memory, else one.
            constexpr int kAhead = (MS * NCB <= 4) ? 2 : 1;
            // first steps of chunk c (b0), c+1 (b1) and c+2 (b2), read one chunk ahead with scalar loads
            int b0 = fetch_int(sp, c_first), b1 = fetch_int(sp, c_first + 1),
                b2 = fetch_int(sp, c_first + 2 < p.n_chunks ? c_first + 2 : p.n_chunks);
            // the first steps of a chunk are requested at the end of the previous chunk's steps, so they arrive
            // while the chunk after it is written to LDS and the workgroup meets at the barrier
            StepRegs<NCB> rg;
            auto prefetch_steps = [&](int c0, int c1) {
                if (active && c0 < c1) {
                    prefetch_first_steps<NCB>(rg, gt, bt, c0, c1, lane);
                } else {                               // defined on every path
#pragma unroll
                    for (int i = 0; i < kIdxAhead; ++i) rg.kk[i] = 0u;
#pragma unroll
                    for (int i = 0; i < prefetch_depth<NCB>(); ++i)
#pragma unroll
                        for (int cb = 0; cb < NCB; ++cb) rg.bq[i][cb] = tw_u16x8{0, 0, 0, 0, 0, 0, 0, 0};
                }
            };
            auto steps_of = [&](int j) {
                const int c = c_first + j;
                if (active && b0 < b1)
                    run_steps<DT, MS, NCB>(acc, rg, smem + (j & 1) * p.abuf_bytes, at_pitch_of<MS>(), gt, bt, b0, b1, lane);
                if (has_ew && active) add_ew_residual<DT, MS, NCB>(p, d.tile, c, acc, smem + (j & 1) * p.abuf_bytes, at_pitch_of<MS>(), lane);
                if constexpr (!SPLIT)
                    if (xbuf != nullptr) xc_chunk<DT, MS>(p, d, c, smem + (j & 1) * p.abuf_bytes, at_pitch_of<MS>(), stage, lane);
                b0 = b1; b1 = b2;
                b2 = fetch_int(sp, c + 3 < p.n_chunks ? c + 3 : p.n_chunks);
                if (j + 1 < n_loc) prefetch_steps(b0, b1); else prefetch_steps(0, 0);
            };
            prefetch_steps(b0, b1);
            if constexpr (SPLIT) {
                commit(first, 0);
                a_zero_row(p, smem, BM, tid);
                a_zero_row(p, smem + p.abuf_bytes, BM, tid);
            }
            if constexpr (kAhead == 1) {
                __syncthreads();
                for (int j = 0; j < n_loc; ++j) {
                    ARegs<AB> ar;
                    issue_or_zero(ar, j + 1);
                    steps_of(j);
                    commit(ar, j + 1);
                    __syncthreads();
                }
            } else {
                // chunk j waits in ring register set j % 2; the loop is unrolled by two so that the sets
                // are addressed statically
                ARegs<AB> ar0, ar1;
                issue_or_zero(ar1, 1);
                __syncthreads();
                for (int j = 0; j < n_loc; j += 2) {
                    issue_or_zero(ar0, j + 2);
                    steps_of(j);
                    commit(ar1, j + 1);
                    __syncthreads();
                    if (j + 1 < n_loc) {
                        issue_or_zero(ar1, j + 3);
                        steps_of(j + 1);
                        commit(ar0, j + 2);
                    }
                    __syncthreads();
                }
            }
            if (active) {
                if constexpr (SPLIT) {
                    dump_partial<MS, NCB>(p.partials + ((((long)part * p.n_mblocks + mb) * p.T + ti) * (long)(MS * NCB * 1024)), acc, lane);
                } else {
                    if (xbuf != nullptr) xc_finish<DT, MS, FUSED, TRANS>(p, d, stage, xbuf, lane);
                    if constexpr (TRANS) store_tile_t<DT, MS, NCB, FUSED>(p, d, acc, stage, dpos, row0, lane, 0, NCB, xbuf);
                    else store_tile<DT, MS, NCB, FUSED>(p, d, acc, stage, dpos, row0, lane, xbuf, xcols);
                }
            }
        }
    }
    };
    if constexpr (MODE == 2) {
        if (wave >= kWaves / 2) run_items(std::integral_constant<int, 2>{});
        else run_items(std::integral_constant<int, 1>{});
    } else {
        run_items(std::integral_constant<int, 0>{});
    }
    // the last workgroup to leave puts the counters back to zero for the next call
    if (tid == 0 && p.n_items > (int)gridDim.x) {
        __threadfence();
        const int done = atomicAdd(&p.counters[1], 1);
        if (done == (int)gridDim.x - 1) {
            atomicExch(&p.counters[0], 0);
            atomicExch(&p.counters[1], 0);
        }
    }
}

// Second kernel of a split-K product.  A workgroup is one wave and takes one piece of one (row block, tile): on the
// row-major boundary one pass of the tile's epilogue (eight rows, all column blocks), on the transposed boundary
// one column block (all 64 tokens).  It adds that piece's partial results of all parts in the order of the parts
// (a fixed order: the result does not depend on which workgroup of the first kernel finished first) and stores it
// through the epilogue of the main kernel (column scatter, zeros of pruned columns, fused bias and activation).
// The pieces are this small because a compute unit brings in only about 16 KB per microsecond from memory (its
// queue of outstanding misses times the latency): a wave that summed a whole tile (32 KB per part) would take as
// long as the chunks it saves.
template <int DT, int NCB, bool FUSED, bool TRANS>
__global__ __launch_bounds__(64) void tw_splitk_reduce_kernel(const TwGemmParams p) {
    constexpr int MS = 2;
    constexpr int SUB = TRANS ? NCB : 4 * MS;               // pieces per tile
    constexpr int NL = TRANS ? 4 * MS : NCB;                // 1 KB loads per piece and part
    __shared__ __attribute__((aligned(16))) unsigned char stage[kStageBytes];
    const int lane = threadIdx.x & 63;
    const int unit = (int)blockIdx.x;                       // ((row block * T) + tile) * SUB + piece
    const int sub = unit % SUB, mt = unit / SUB;
    const int mb = mt / p.T, ti = mt - mb * p.T;
    const int row0 = mb * p.row_step;
    const long part_stride = (long)p.n_mblocks * p.T * (MS * NCB * 1024);
    const float* src = p.partials + ((long)mb * p.T + ti) * (long)(MS * NCB * 1024) + lane * 4;
    // load i of the piece: row-major (ms, q) = sub, cb = i; transposed cb = sub, (ms, q) = i
    int off[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int msq = TRANS ? i : sub, cb = TRANS ? sub : i;
        off[i] = (((msq >> 2) * NCB + cb) * 4 + (msq & 3)) * 256;
    }
    // The first parts (as many as a hundred registers or so hold: 8 with four loads to a piece, 12 with two, 16 with one, 5 on the
    // transposed boundary with eight) are requested before anything waits, for the tile's descriptor or for one of them;
    // further parts follow in batches.  Past the last part the last one is requested again, from the caches, and not
    // added (branches around those requests cost more than they do; half as many requests go out for half as many parts).
    // Two parts at a time, a round trip to memory for every two: 3072 -> 768 at 64 / 512 rows 12.3 / 17.4 us, this way 11.0 /
    // 16.7, transposed 4608 -> 500 at 100 tokens 13.7, this way 11.3.
    constexpr int kFirst = TRANS ? 5 : NL == 4 ? 8 : NL == 2 ? 12 : 16, kAhead = TRANS ? 4 : 7;
    tw_f32x4 s[NL];
    TileU d;
    unsigned dpos[NCB];
    float col[NCB];
    auto fetch_columns = [&] {
        d = fetch_tile(p, ti);
        const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) dpos[cb] = dp[cb];
    };
    if constexpr (FUSED) fetch_columns();                   // (the bias follows from them: they must not wait for the parts)
    auto first_parts = [&](auto batch) {
        constexpr int B = decltype(batch)::value;
        tw_f32x4 v[B][NL];
#pragma unroll
        for (int a = 0; a < B; ++a) {
            const int from = a < p.n_parts ? a : p.n_parts - 1;
#pragma unroll
            for (int i = 0; i < NL; ++i) v[a][i] = *(const tw_f32x4*)(src + from * part_stride + off[i]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FUSED) fetch_col_bias<DT, NCB>(p, d, dpos, col);
        else fetch_columns();
#pragma unroll
        for (int i = 0; i < NL; ++i) s[i] = v[0][i];
#pragma unroll
        for (int a = 1; a < B; ++a)
            if (a < p.n_parts) {                            // wave-uniform
#pragma unroll
                for (int i = 0; i < NL; ++i) s[i] += v[a][i];
            }
    };
    if (p.n_parts <= (kFirst + 1) / 2) first_parts(std::integral_constant<int, (kFirst + 1) / 2>{});
    else first_parts(std::integral_constant<int, kFirst>{});
    for (int part = kFirst; part < p.n_parts; part += kAhead) {
        tw_f32x4 v[kAhead][NL];
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
            const int from = part + a < p.n_parts ? part + a : p.n_parts - 1;
#pragma unroll
            for (int i = 0; i < NL; ++i) v[a][i] = *(const tw_f32x4*)(src + from * part_stride + off[i]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < kAhead; ++a)
            if (part + a < p.n_parts) {                     // wave-uniform
#pragma unroll
                for (int i = 0; i < NL; ++i) s[i] += v[a][i];
            }
    }
    if constexpr (FUSED) {
        float b[NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            b[i] = TRANS ? 0.f : col[TRANS ? 0 : i];
            if constexpr (TRANS) {
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) b[i] = cb == sub ? col[cb] : b[i];
            }
        }
        apply_bias_act4<NL>(s, b, p.act);
    }
    tw_f32x16 acc[MS][NCB];
    zero_acc<MS, NCB>(acc);
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int msq = 4 * ms + q;
                if ((TRANS ? cb : msq) == sub) {            // wave-uniform
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[ms][cb][4 * q + e] = s[TRANS ? msq : cb][e];
                }
            }
    if constexpr (TRANS) store_tile_t<DT, MS, NCB, FUSED, true>(p, d, acc, stage, dpos, row0, lane, sub, sub + 1);
    else store_tile<DT, MS, NCB, FUSED, true>(p, d, acc, stage, dpos, row0, lane, nullptr, nullptr, sub, sub + 1);
}

// The sums of a team's waves for PER units of a tile, in the order of the waves.  `piece`: the first wave's first piece of the
// first unit; the pieces of a unit lie 4 KB (row-major: a column block on) or 1 KB (transposed: eight rows on) apart, the units
// 1 KB or 4 KB, the waves NCB * 4 KB.  All pieces are read before the first is added (one wave's piece after another's is up
// to 28 round trips to LDS: 60 -> 961 (G = 128) at 2156 rows 9.3 us, this way 8.4).
template <int TEAM, int PER, int NL, bool TRANS, int NCB>
__device__ __forceinline__ void team_sum(const unsigned char* piece, tw_f32x4 (&sum)[PER][NL]) {
    tw_f32x4 v[TEAM][PER][NL];
#pragma unroll
    for (int i = 0; i < TEAM; ++i)
#pragma unroll
        for (int k = 0; k < PER; ++k)
#pragma unroll
            for (int l = 0; l < NL; ++l)
                v[i][k][l] = *(const tw_f32x4*)(piece + i * (NCB * 4096) + k * (TRANS ? 4096 : 1024) + l * (TRANS ? 1024 : 4096));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < PER; ++k)
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            sum[k][l] = v[0][k][l];
#pragma unroll
            for (int i = 1; i < TEAM; ++i) sum[k][l] += v[i][k][l];
        }
}

// K resident, row blocks of 32, few tiles per workgroup: a TEAM of 8, 4 or 2 waves shares a tile.
// With few row blocks a workgroup of the kernel above has one to four tiles for its eight waves, and a launch takes as
// long as one wave takes for its chain: item number, descriptor, A, K indices, a heavy tile's steps one after the other (24
// steps, 3 requests of packed weights ahead), the epilogue.  Here the workgroup's number is its item (a launch is one round of
// workgroups), a wave takes 1 / team of its tile's steps and requests their first operands BEFORE it waits for A,
// and the fp32 sums meet in LDS: every wave leaves its own there, and pass by pass (column block by column block on
// the transposed boundary) the team's waves add them in the order of the steps and store their share of the tile.
// The order of the sums depends on the plan only, so repeated calls are bit-identical.
template <int DT, int NCB, bool FUSED, bool TRANS>
__global__ __launch_bounds__(kThreads) void tw_team_kernel(const TwGemmParams p) {
    constexpr int MS = 1;
    constexpr bool PAIR = kPairResident;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int team = 1 << p.team_shift;
    const int mb = (int)blockIdx.x / p.n_seg, seg = (int)blockIdx.x - mb * p.n_seg;
    const int row0 = mb * p.row_step;
    const int member = wave & (team - 1);
    const int ti = seg + (wave >> p.team_shift) * p.n_seg;
    const bool active = ti < p.T;                            // wave-uniform
    const TileU d = fetch_tile(p, active ? ti : 0);
    const int s0 = (d.nsteps * member) >> p.team_shift, s1 = (d.nsteps * (member + 1)) >> p.team_shift;
    const bool steps = active && s0 < s1;
    const unsigned char* goff = p.blob + p.off_goff + (long)d.first_step * 32;
    const unsigned char* bvals = p.blob + p.off_bvals + (long)d.first_step * NCB * 1024;
    unsigned dpos[NCB];
    StepRegs<NCB> rg;
    auto first_operands = [&] {
        const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) dpos[cb] = dp[cb];
        prefetch_first_steps<NCB>(rg, goff, bvals, steps ? s0 : 0, steps ? s1 : 1, lane);
    };
    // A in one batch where it is short (768 columns), else in batches of twelve requests
    auto stage_a = [&](auto batch) {
        constexpr int B = decltype(batch)::value;
        const int tasks = TRANS ? at_tasks<MS>(p.K) : a_tasks<MS, PAIR>(p.K);
        constexpr int per = kWaves * (TRANS || !PAIR ? B : B / 2);
        for (int t0 = wave; t0 < tasks || t0 == wave; t0 += per) {
            ARegs<B> ar;
            if constexpr (TRANS) at_issue<MS, B>(p, ar, row0, 0, p.K, t0, lane);
            else a_issue<MS, B, PAIR>(p, ar, row0, 0, p.K, t0, lane);
            if (t0 == wave) first_operands();
            if constexpr (TRANS) at_commit<MS, B>(p, ar, smem, p.K, t0, lane);
            else a_commit<MS, B, PAIR>(p, ar, smem, p.K, t0, lane);
        }
    };
    if (p.K <= 768) stage_a(std::integral_constant<int, 6>{});
    else stage_a(std::integral_constant<int, 12>{});
    a_zero_row(p, smem, 32 * MS, tid);
    __syncthreads();
    tw_f32x16 acc[MS][NCB];
    zero_acc<MS, NCB>(acc);
    if (steps) run_steps<DT, MS, NCB>(acc, rg, smem, at_pitch_of<MS>(), goff, bvals, s0, s1, lane);
    __syncthreads();                                         // everyone is done with A: the sums take its place
    unsigned char* sums = smem + wave * (NCB * 4096);        // piece (cb, q) of a wave: 1 KB, 16 bytes a lane
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *(tw_f32x4*)(sums + (cb * 4 + q) * 1024 + lane * 16) =
                tw_f32x4{acc[0][cb][4 * q], acc[0][cb][4 * q + 1], acc[0][cb][4 * q + 2], acc[0][cb][4 * q + 3]};
    __syncthreads();
    float col[NCB];
    if constexpr (FUSED) fetch_col_bias<DT, NCB>(p, d, dpos, col);
    // this wave's share: passes u0 .. u1 of eight rows (four in all), or column blocks on the transposed boundary
    constexpr int UNITS = TRANS ? NCB : 4;
    const int per = (UNITS + team - 1) >> p.team_shift;
    const int u0 = member * per, u1 = u0 + per < UNITS ? u0 + per : UNITS;
    constexpr int NL = TRANS ? 4 : NCB;                      // pieces of a unit
    const unsigned char* first = smem + (wave - member) * (NCB * 4096) + lane * 16;
    auto add_up = [&](auto team_size) {
        constexpr int TEAM = decltype(team_size)::value, PER = (UNITS + TEAM - 1) / TEAM;
        tw_f32x4 v[PER][NL];
        if (u0 < UNITS) team_sum<TEAM, PER, NL, TRANS, NCB>(first + u0 * (TRANS ? 4096 : 1024), v);
        if constexpr (FUSED) {
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                float b[NL];
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    b[l] = col[TRANS ? 0 : l];
                    if constexpr (TRANS) {
#pragma unroll
                        for (int cb = 1; cb < NCB; ++cb) b[l] = cb == u0 + k ? col[cb] : b[l];
                    }
                }
                apply_bias_act4<NL>(v[k], b, p.act);
            }
        }
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int k = 0; k < PER; ++k)
                    if ((TRANS ? cb : q) == u0 + k) {        // wave-uniform
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[0][cb][4 * q + e] = v[k][TRANS ? q : cb][e];
                    }
    };
    if (team == 8) add_up(std::integral_constant<int, 8>{});
    else if (team == 4) add_up(std::integral_constant<int, 4>{});
    else add_up(std::integral_constant<int, 2>{});
    __syncthreads();                                         // the staging areas of the epilogue lie over the sums
    if (!active || u0 >= u1) return;
    unsigned char* stage = smem + p.stage_off + wave * kStageBytes;
    if constexpr (TRANS) store_tile_t<DT, MS, NCB, FUSED, true>(p, d, acc, stage, dpos, row0, lane, u0, u1);
    else store_tile<DT, MS, NCB, FUSED, true>(p, d, acc, stage, dpos, row0, lane, nullptr, nullptr, u0, u1);
}

// ---- transposed boundary, one tile of one block of tokens per workgroup ----
// The kernels above bring a block of At into LDS once and gather from it for every tile; what a compute unit then streams is
// the packed weights of ALL tiles per 64 tokens.  With the activations transposed there is another way: the K rows that ONE tile
// keeps are whole rows of the block (256 or 512 bytes), so they can be fetched straight into LDS in the order of the tile's
// contraction slots, and the product of a tile and a token block is an ordinary dense one: nothing is staged through
// registers, no row that the tile does not keep is read, and the main loop reads LDS at fixed addresses.
//
// A workgroup is four waves, its block 128 tokens (tiles of four column blocks, two waves side by side) or 256 (narrower tiles); a
// wave multiplies 64 tokens x 64 (32) columns in the order of the tile's steps, which is the order of the kernels above: both
// boundaries give the same bits.  A ring of kRowsStages stages of one step (16 slots) is filled by direct loads.  Several workgroups share a
// compute unit, so one's first loads and stores pass while others multiply: with four stages four while LDS holds them (40 KB each: tiles
// of up to 123 steps with G = 128 and up to 59 with G = 32), else three (G = 64, whose four stages alone take 40 KB, up to 208 steps; G = 128
// up to 336, G = 32 up to 272), else two.  (Registers allow four.)
//
// LDS row r of a stage is slot position r of the step's list (off_goff); its 16-byte pieces are kept at piece ^ 4 * (r / 2 % 4): a
// transposing read takes four rows r, r + 2, r + 4, r + 6 at the same tokens, which then lie in different banks.
// Padded slots, tokens past M and steps past the end are offsets out of the descriptor's range: they fetch zeros.
//
// What bounds it: full batches the compute unit's loads (8 KB a step, about 110 ns with four workgroups in their main loops, of which the 110 to
// 120 KB/us that a compute unit reads from the L2 are 70; its address and data units are busy 53 and 64 % of 16384 x 768 -> 3072), two
// workgroups or fewer the latency of a stage, 170 ns a step with four stages on their way, 125 with eight (8192 x 4096 -> 1024: no unit
// is busy more than 36 % of the launch).  What the compiler loads itself is consumed before the first direct load: its waits do not know of those, and a
// wait for one of its own behind them drained the ring (16384 tokens of 768 -> 3072 41.2 us, now 34.0).
// Before (a resident or streamed block of 64 tokens, all tiles) -> now: 16384 tokens of 768 -> 3072 39.3 -> 34.0 us, 8192 of
// 4096 -> 1024, skewed 42.2 -> 28.1 (its heaviest tile has 159 steps), 84745 of 1152 -> 130 (G = 32) 105 -> 34, 54959 of
// 576 -> 201 51 -> 14.
//
// Workgroups of one XCD (ids equal modulo 8) share its L2: the token blocks are dealt out to the XCDs, rows_group blocks at a
// time, as many as leave the rows of those of one XCD in its L2; within a group the tiles that keep the most rows go first.  A group is a multiple of
// eight blocks, so that a block stays with its XCD from tile to tile (77 blocks in one group, 19648 tokens of 571 -> 2289, G = 32:
// 112 us); up to seven blocks that are left over go first, whichever XCDs they meet.
template <int NCB> constexpr int rows_bt() { return NCB == 4 ? 128 : 256; }
template <int NCB> constexpr int rows_stage_bytes() { return rows_bt<NCB>() * 32 + NCB * 1024; }
constexpr unsigned kRowsRange = 0x40000000u;               // (twice that is out of range as well)
constexpr int kRowsStoreArea = 32 * (64 * 2 + 8);
static_assert(4 * kRowsStoreArea <= 4 * rows_stage_bytes<4>() && 4 * kRowsStoreArea <= 4 * rows_stage_bytes<1>(),
              "the epilogue's staging areas lie over the ring");

template <int DT, int NCB, bool FUSED, int kRowsStages>
__global__ __launch_bounds__(256, kRowsStages == 4 ? 4 : 2) void tw_rows_kernel(const TwGemmParams p) {
    constexpr int BT = rows_bt<NCB>(), CB = NCB == 4 ? 2 : NCB, IA = BT / 128, STAGE = rows_stage_bytes<NCB>(), A_BYTES = BT * 32;
    constexpr int kLoads = IA + 1;                           // requests of a wave per stage
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int wt = NCB == 4 ? wave >> 1 : wave, wc = NCB == 4 ? wave & 1 : 0;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // the item: tile number t (0: the heaviest), token block mb
    const int odd = p.n_mblocks & 7, id = (int)blockIdx.x - odd * p.T;       // (id < 0: one of the odd blocks)
    const int per = p.rows_group * p.T, g = id < 0 ? 0 : id / per, rem = id < 0 ? (int)blockIdx.x : id - g * per;
    const int block0 = id < 0 ? 0 : odd + g * p.rows_group, left = p.n_mblocks - block0;
    const int width = id < 0 ? odd : left < p.rows_group ? left : p.rows_group;
    const int t = rem / width, m0 = (block0 + rem - t * width) * BT;
    // (with K resident the dispatch order puts the lightest kWaves tiles, lightest first, in front of the others)
    const bool light_first = p.n_chunks == 1 && p.T > kWaves;
    const TileU d = fetch_tile(p, !light_first ? t : t < p.T - kWaves ? t + kWaves : p.T - 1 - t);

    auto descriptor = [](const void* base, unsigned bytes) {
        const uint64_t b = (uint64_t)base;
        return tw_u32x4{(unsigned)uni((int)(unsigned)b), (unsigned)uni((int)(unsigned)(b >> 32)) & 0xFFFFu, bytes, 0x00020000u};
    };
    const tw_u32x4 da = descriptor(p.A + m0, kRowsRange);
    const tw_u32x4 db = descriptor(p.blob + p.off_bvals + (long)d.first_step * NCB * 1024, (unsigned)d.nsteps * (NCB * 1024u));
    const unsigned lda2 = 2u * (unsigned)p.lda;

    // What this lane fetches: request n of a stage brings row 4*wave + 2*n + its share of the wave's 4 / IA rows, and of that
    // row the 16-byte piece that belongs at its place in LDS.
    constexpr int kSlots = BT / 8;                           // pieces of a row
    const int frow = 4 * wave + lane / kSlots;
    auto swz = [](int r) { return ((r >> 1) & 3) << 2; };
    unsigned a_off[IA];
#pragma unroll
    for (int n = 0; n < IA; ++n) {
        const int piece = (lane % kSlots) ^ swz(frow + 2 * n);
        a_off[n] = m0 + piece * 8 < p.M ? (unsigned)piece * 16u : kRowsRange;
    }
    const bool b_lane = lane < NCB * 16;
    unsigned b_off = (unsigned)(wave * NCB * 256 + (lane & (NCB * 16 - 1)) * 16);   // of the step the cursor stands on
    // Where the rows of the tile's slots lie: byte offset in At, kRowsRange for a padded slot and behind the last step.  The list
    // waits in LDS behind the ring; the lanes work out those of the first stages themselves.
    const unsigned short* goff = (const unsigned short*)(p.blob + p.off_goff + (long)d.first_step * 32);
    unsigned* const list = (unsigned*)(smem + kRowsStages * STAGE);
    int ends = 0;                                            // K streamed: lane l holds where chunk l's steps end
    if (p.n_chunks > 1) ends = ((const int*)(p.blob + p.off_step_ptr))[d.step_ptr + 1 + (lane < p.n_chunks ? lane : p.n_chunks - 1)];
    unsigned short first[kRowsStages][IA];
#pragma unroll
    for (int i = 0; i < kRowsStages; ++i)
#pragma unroll
        for (int n = 0; n < IA; ++n) first[i][n] = goff[(i < d.nsteps ? i : d.nsteps - 1) * 16 + frow + 2 * n];
    const int n_list = 16 * (d.nsteps + kRowsStages + 1);    // (what is read of it: one step past the end)
    auto slot_row = [&](int i) { return goff[i < 16 * d.nsteps ? i : 0]; };
    unsigned short ahead[2];                                 // two slots of a thread cover 32 steps
#pragma unroll
    for (int n = 0; n < 2; ++n) ahead[n] = slot_row(16 * kRowsStages + tid + 256 * n);
    unsigned dpos[CB];
    {
        const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB + wc * CB;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) dpos[cb] = dp[cb];
    }
    auto row_of = [&](int step, unsigned k) {                // k: chunk-local row as the blob has it
        unsigned base = 0;
        for (int c = 0; c + 1 < p.n_chunks; ++c) base += step >= __builtin_amdgcn_readlane(ends, c) ? (unsigned)p.k_chunk : 0u;
        return step < d.nsteps && k != (unsigned)p.k_chunk ? __umul24(base + k, lda2) : kRowsRange;
    };
    auto issue = [&](unsigned buf, const unsigned (&row)[IA]) {     // buf: LDS address of the stage
#pragma unroll
        for (int n = 0; n < IA; ++n) tw_load_lds<false>(da, row[n] + a_off[n], buf + (unsigned)(wave * IA + n) * 1024u);
        if (NCB == 4 || b_lane) tw_load_lds<false>(db, b_off, buf + A_BYTES + (unsigned)(wave * NCB) * 256u);
        b_off += NCB * 1024u;
    };
    // (in front of the direct loads: the compiler does not count those and would wait for them with its own)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int i = 16 * kRowsStages + tid + 256 * n;
        if (i < n_list) list[i] = row_of(i >> 4, ahead[n]);
    }
    unsigned kk[IA];
#pragma unroll
    for (int i = 0; i < kRowsStages; ++i) {
#pragma unroll
        for (int n = 0; n < IA; ++n) kk[n] = row_of(i, first[i][n]);
        issue(lds0 + i * STAGE, kk);
    }
    for (int i = 16 * kRowsStages + 512 + tid; i < n_list; i += 256) list[i] = row_of(i >> 4, slot_row(i));
    const unsigned* rows = list + 16 * kRowsStages + frow;   // of the step the cursor stands on
    EpiBias<CB> eb;
    if constexpr (FUSED) fetch_col_bias<DT, CB>(p, d, dpos, eb.col);

    // where this lane's operands lie in a stage (see run_steps for the lanes of a transposing read)
    const int h = lane >> 5, j = lane & 15, q = j >> 2;
    const unsigned oa = (unsigned)(8 * h + 2 * q) * (BT * 2) +
                        (unsigned)(((wt * 8 + ((lane >> 4) & 1) * 2 + ((j & 3) >> 1)) ^ (q << 2)) * 16 + (j & 1) * 8);
    const unsigned ob = (unsigned)(A_BYTES + wc * CB * 1024 + lane * 16);
    tw_f32x16 acc[2][CB];
    zero_acc<2, CB>(acc);
    tw_u16x8 a[2][2], b[2][CB];
    auto fetch = [&](int slot, int cur) {                    // operands of the step in stage `cur` (constants)
        const unsigned char* st = smem + cur * STAGE;
#pragma unroll
        for (int ms = 0; ms < 2; ++ms) {
            const tw_i16x4 lo = tw_lds_read_tr(st + (oa ^ (unsigned)(ms * 64)));
            const tw_i16x4 hi = tw_lds_read_tr(st + (oa ^ (unsigned)(ms * 64)) + BT * 2);
            a[slot][ms] = tw_u16x8{(unsigned short)lo[0], (unsigned short)lo[1], (unsigned short)lo[2], (unsigned short)lo[3],
                                   (unsigned short)hi[0], (unsigned short)hi[1], (unsigned short)hi[2], (unsigned short)hi[3]};
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) b[slot][cb] = *(const tw_u16x8*)(st + ob + cb * 1024);
    };
    auto fetch_rows = [&] {
#pragma unroll
        for (int n = 0; n < IA; ++n) kk[n] = rows[2 * n];
        rows += 16;
    };
    // A step: when the next step's stage has landed and every wave has this step's operands in registers, this step's stage is
    // refilled and the next operands are read, behind this step's products.
    auto step = [&](int cur) {                               // stage `cur` of the ring (a constant)
        tw_lds_wait<(kRowsStages - 2) * kLoads>();
        issue(lds0 + (unsigned)cur * STAGE, kk);
        fetch((cur + 1) & 1, (cur + 1) % kRowsStages);
        fetch_rows();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int ms = 0; ms < 2; ++ms) acc[ms][cb] = tw_mfma<DT>(a[cur & 1][ms], b[cur & 1][cb], acc[ms][cb]);
        __builtin_amdgcn_sched_barrier(0);
    };
    tw_lds_wait<(kRowsStages - 1) * kLoads>();
    fetch(0, 0);
    fetch_rows();
    int s = 0;
    for (; s + kRowsStages <= d.nsteps; s += kRowsStages) {
#pragma unroll
        for (int i = 0; i < kRowsStages; ++i) step(i);
    }
#pragma unroll
    for (int i = 0; i < kRowsStages - 1; ++i)
        if (s + i < d.nsteps) step(i);
    tw_lds_wait<0>();                                        // nothing on its way into the ring any more: the staging areas lie over it
    if constexpr (FUSED) apply_bias_act<2, CB>(acc, eb, p.act);
    store_tile_t<DT, 2, CB, FUSED, true>(p, d, acc, smem + wave * kRowsStoreArea, dpos, m0 + wt * 64, lane, 0, CB, nullptr, wc == 0);
}

// ---- row-major boundary, K streamed, at most four tiles of a row block per workgroup ----
// As MODE 2 above: four waves multiply, four bring in chunks of 384 columns of 64 rows, K-major and double-buffered, one barrier per
// chunk.  The loading waves hold nothing in registers: direct loads bring windows of 64 columns into a ring of kWindows
// windows as they lie in memory, always that many on their way, into the next item too; a wave turns the 16 rows of a window that it
// has asked for itself (no barrier there) with transposing LDS reads, 4 rows x 16 columns a quarter wave, and writes the four
// rows of a column in one piece.  MODE 2 keeps a chunk in registers and writes every value by itself (96 2-byte
// writes of a wave for a chunk, 24 8-byte ones here).
// The barriers are the instruction itself: __syncthreads() would also wait for the packed weights asked for ahead.
// What bounds it now are the multiplying waves.  100352 x 2304 -> 256 (G = 64, bias, ReLU) 151.6 -> 138 us; bringing A in and turning it
// alone takes 73 (6.3 TB/s), with the epilogue 95, the steps and the epilogue alone 91: an item's heaviest tile is one wave's,
// and the loading waves stop two chunks ahead of an epilogue.  28367 x 1576 -> 512 57 -> 42 us, 12658 x 2625 -> 960 67 -> 48,
// 20335 x 4292 -> 256 87 -> 62, 7936 x 1668 -> 256 24.3 -> 16.4; 5400 random calls with 1500 rows and more 1.25 times as fast on average, 37
// slower by more than 2 %, the worst by 9 % (three or four wide tiles; 77094 x 4957 -> 459 321 us before, 350 now).  (29 to 36 scalar registers
// spill into vector ones: the loading and the multiplying waves' constants in one kernel.  The counters agree: a compute unit's queue of
// misses is full for 44 % of the convolution's launch, the waves wait 14 % of their time.)
// Tried without gain: two waves a tile with 32 rows each (155 us), first operands asked for across chunks (branches between
// the steps cost more), row-major chunks with 2-byte gathers (171), four waves that share a tile in place of split K.
//
// 16-byte piece c of row r of a window lies at slot c ^ (r % 8) of the row.
constexpr int kStreamChunk = TW_K_STREAM_CHUNK, kWindow = 64, kWindows = 4, kStreamLoaders = 4, kStreamTiles = 4;
constexpr unsigned kWindowBytes = 64 * kWindow * 2;
constexpr unsigned kStreamRange = 0x80000000u;
static_assert(kStreamChunk % kWindow == 0, "whole windows");

template <int DT, int NCB, bool FUSED>
__global__ __launch_bounds__(kThreads) void tw_stream_kernel(const TwGemmParams p) {
    constexpr unsigned PITCH = at_pitch_of<2>();
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int grid = (int)gridDim.x;

    if (wave >= kStreamTiles) {
        const int lw = wave - kStreamTiles;                  // rows 16 lw .. of a block
        unsigned char* const ring = smem + p.urow_off + lw * 2048;
        const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
        const unsigned lda2 = 2u * (unsigned)p.lda;
        if (lw == 0) {                                       // what padded slots read: row k_chunk of both buffers
            if (lane < 32) *(unsigned*)(smem + (unsigned)kStreamChunk * PITCH + lane * 4) = 0u;
            else *(unsigned*)(smem + p.abuf_bytes + (unsigned)kStreamChunk * PITCH + (lane - 32) * 4) = 0u;
        }
        // the request cursor: window cw of chunk cc of item ci, into slot cq of the ring; windows on their way
        int ci = (int)blockIdx.x, cc = 0, cw = 0, cq = 0, ahead = 0;
        const int frow = 16 * lw + (lane >> 3), piece = (lane & 7) ^ (lane >> 3);
        const unsigned foff = (unsigned)frow * lda2 + (unsigned)piece * 16u;
        auto issue = [&] {
            if (ci >= p.n_items) return;
            const int set = ci / p.n_mblocks, row0 = (ci - set * p.n_mblocks) * p.row_step, col0 = cc * kStreamChunk + cw * kWindow;
            const uint64_t base = (uint64_t)(p.A + (long)row0 * p.lda + col0);
            const tw_u32x4 da{(unsigned)uni((int)(unsigned)base), (unsigned)uni((int)(unsigned)(base >> 32)) & 0xFFFFu, kStreamRange, 0x00020000u};
            const int rows = block_end(p, row0) - row0;
            const bool col = col0 + piece * 8 < p.K;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned off = col && frow + 8 * i < rows ? foff + (unsigned)(8 * i) * lda2 : kStreamRange;
                const unsigned to = lds0 + (unsigned)cq * kWindowBytes + (unsigned)i * 1024u;
                if (p.n_seg == 1) tw_load_lds<true>(da, off, to);    // (streaming where nobody else reads these rows: see load_a16)
                else tw_load_lds<false>(da, off, to);
            }
            cq = (cq + 1) & (kWindows - 1);
            ++ahead;
            if (++cw == kStreamChunk / kWindow || col0 + kWindow >= p.K) {
                cw = 0;
                if (++cc == p.n_chunks) { cc = 0; ci += grid; }
            }
        };
#pragma unroll
        for (int i = 0; i < kWindows; ++i) issue();
        const int grp = lane >> 4, j = lane & 15, trow = 4 * grp + (j >> 2);
        const unsigned from = (unsigned)(trow * 128 + ((((j & 3) >> 1) ^ (trow & 7)) << 4) + (j & 1) * 8);
        const unsigned to = (unsigned)j * PITCH + (unsigned)(16 * lw + 4 * grp) * 2u;
        int q = 0;
        unsigned buf = 0;
        for (int item = (int)blockIdx.x; item < p.n_items; item += grid) {
            for (int c = 0; c < p.n_chunks; ++c) {
                const int width = p.K - c * kStreamChunk, windows = width >= kStreamChunk ? kStreamChunk / kWindow : (width + kWindow - 1) / kWindow;
                for (int w = 0; w < windows; ++w) {
                    if (ahead == kWindows) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * (kWindows - 1)) : "memory");
                    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    const unsigned char* src = ring + (unsigned)q * kWindowBytes;
                    unsigned char* dst = smem + buf + to + (unsigned)(w * kWindow) * PITCH;
                    tw_i16x4 v[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = tw_lds_read_tr(src + (from ^ (unsigned)(t << 5)));
#pragma unroll
                    for (int t = 0; t < 4; ++t) *(tw_u32x2*)(dst + t * 16 * PITCH) = __builtin_bit_cast(tw_u32x2, v[t]);
                    q = (q + 1) & (kWindows - 1);
                    --ahead;
                    issue();                                 // (the reads of this slot are over: their values have been written)
                }
                tw_lds_wait<63>();                           // the chunk is there
                buf = buf == 0 ? p.abuf_bytes : 0u;
            }
        }
        return;
    }

    unsigned char* stage = smem + p.stage_off + wave * kStageBytes;
    unsigned buf = 0;
    for (int item = (int)blockIdx.x; item < p.n_items; item += grid) {
        const int set = item / p.n_mblocks, row0 = (item - set * p.n_mblocks) * p.row_step;
        const int ti = set * p.tiles_per_set + wave;
        const bool active = wave < p.tiles_per_set && ti < p.T;              // wave-uniform
        const TileU d = fetch_tile(p, active ? ti : 0);
        const int* sp = (const int*)(p.blob + p.off_step_ptr) + d.step_ptr;
        unsigned dpos[NCB];
        {
            const unsigned* dp = (const unsigned*)(p.blob + p.off_dpos) + ((long)d.tile * 32 + (lane & 31)) * NCB;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) dpos[cb] = dp[cb];
        }
        tw_f32x16 acc[2][NCB];
        zero_acc<2, NCB>(acc);
        const unsigned char* gt = p.blob + p.off_goff + (long)d.first_step * 32;
        const unsigned char* bt = p.blob + p.off_bvals + (long)d.first_step * NCB * 1024;
        int s0 = 0, s1 = fetch_int(sp, 1), s2 = fetch_int(sp, p.n_chunks < 2 ? p.n_chunks : 2);
        for (int c = 0; c < p.n_chunks; ++c) {
            const bool steps = active && s0 < s1;
            StepRegs<NCB> rg;
            if (steps) prefetch_first_steps<NCB>(rg, gt, bt, s0, s1, lane);
            tw_lds_wait<63>();
            if (steps) run_steps<DT, 2, NCB>(acc, rg, smem + buf, PITCH, gt, bt, s0, s1, lane);
            s0 = s1;
            s1 = s2;
            s2 = fetch_int(sp, c + 3 < p.n_chunks ? c + 3 : p.n_chunks);
            buf = buf == 0 ? p.abuf_bytes : 0u;
        }
        if (active) store_tile<DT, 2, NCB, FUSED>(p, d, acc, stage, dpos, row0, lane);
    }
}

// First kernel of a split-K product, row-major boundary (MODE 3 above for everything else): a workgroup has one item (part, tile set, row
// block) and few chunks, so nothing overlaps its first operands and few tiles leave waves without work.  All eight waves
// bring in A: direct loads put chunks as they lie in memory into two buffers, both on their way at once; a wave turns the eight rows that it
// has asked for itself into the K-major copy, as in tw_stream_kernel (8 rows x 32 columns a reading instruction).  And a tile has 8 / tiles
// of the waves: two row halves (H = 2, up to four tiles) and two column halves (CG = 2, up to two tiles of 64 or 128 columns).
// The results are those of MODE 3, bit for bit.
// What bounds it is the chain of one part: launch, a chunk's latency, the heaviest tile's steps, the dump (32 KB a tile and part).  MODE 3
// -> this kernel, whole calls: 2048 x 3072 -> 768 23.6 -> 22.6 us, 1745 x 3441 -> 477 26.6 -> 21.7, 348 x 2002 -> 746 16.0 -> 13.6,
// 64 x 2593 -> 1549 with GELU 14.8 -> 12.4; 4990 random split calls 1.23 times as fast on average (0.95 to 1.5).
template <int DT, int NCB, int H, int CG>
__global__ __launch_bounds__(kThreads) void tw_part_kernel(const TwGemmParams p) {
    constexpr unsigned PITCH = at_pitch_of<2>(), RAW = 64 * kStreamChunk * 2, WIN = 1024;      // a wave's window: 8 rows x 64 columns
    constexpr int kWin = kStreamChunk / kWindow, MS = 2 / H, NC = NCB / CG;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int item = (int)blockIdx.x;
    const int sp_item = item / p.n_mblocks, mb = item - sp_item * p.n_mblocks;
    const int part = sp_item / p.n_seg, set = sp_item - part * p.n_seg;
    const int c_first = part * p.chunks_per_part;
    const int n_loc = (p.n_chunks - c_first) < p.chunks_per_part ? (p.n_chunks - c_first) : p.chunks_per_part;
    const int row0 = mb * 64;

    unsigned char* const raw = smem + p.abuf_bytes + wave * (kWin * WIN);                      // this wave's rows of buffer 0
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)raw;
    const unsigned lda2 = 2u * (unsigned)p.lda;
    const int frow = 8 * wave + (lane >> 3), piece = (lane & 7) ^ (lane >> 3);
    auto issue = [&](int j) {                                // chunk j of the part
        const int col0 = (c_first + j) * kStreamChunk;
        const uint64_t base = (uint64_t)(p.A + (long)row0 * p.lda + col0);
        const tw_u32x4 da{(unsigned)uni((int)(unsigned)base), (unsigned)uni((int)(unsigned)(base >> 32)) & 0xFFFFu, kStreamRange, 0x00020000u};
        const bool row = row0 + frow < p.M;
#pragma unroll
        for (int w = 0; w < kWin; ++w)
            tw_load_lds<false>(da, row && col0 + w * kWindow + piece * 8 < p.K ? (unsigned)frow * lda2 + (unsigned)(w * 128 + piece * 16) : kStreamRange,
                               lds0 + (unsigned)(j & 1) * RAW + (unsigned)w * WIN);
    };
    const int slot = wave / (H * CG), half = wave % H, cg = (wave / H) % CG;
    const int ti = set * p.tiles_per_set + slot;
    const bool active = slot < p.tiles_per_set && ti < p.T;
    issue(0);
    if (n_loc > 1) issue(1);
    const TileU d = fetch_tile(p, active ? ti : 0);
    const int* sp = (const int*)(p.blob + p.off_step_ptr) + d.step_ptr + c_first;
    const unsigned char* gt = p.blob + p.off_goff + (long)d.first_step * 32;
    const unsigned char* bt = p.blob + p.off_bvals + ((long)d.first_step * NCB + cg * NC) * 1024;
    if (tid < 32) *(unsigned*)(smem + (unsigned)kStreamChunk * PITCH + tid * 4) = 0u;
    int s0 = fetch_int(sp, 0), s1 = fetch_int(sp, 1);
    tw_f32x16 acc[MS][NC];
    zero_acc<MS, NC>(acc);
    // turning: group lane / 16: rows 4 * (group % 2) .. + 3, columns 16 * (group / 2) .. + 15 of 32
    const int j16 = lane & 15, trow = 4 * ((lane >> 4) & 1) + (j16 >> 2), tcol = 16 * (lane >> 5);
    const unsigned from = (unsigned)(trow * 128 + ((((tcol >> 3) + ((j16 & 3) >> 1)) ^ trow) << 4) + (j16 & 1) * 8);
    unsigned char* const to = smem + (unsigned)(tcol + j16) * PITCH + (unsigned)(8 * wave + 4 * ((lane >> 4) & 1)) * 2u;
    for (int j = 0; j < n_loc; ++j) {
        if (j + 1 < n_loc) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(kWin) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const unsigned char* src = raw + (unsigned)(j & 1) * RAW;
#pragma unroll
        for (int w = 0; w < kWin; ++w) {
            tw_i16x4 v[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) v[t] = tw_lds_read_tr(src + w * WIN + (from ^ (unsigned)(t << 6)));
#pragma unroll
            for (int t = 0; t < 2; ++t) *(tw_u32x2*)(to + (unsigned)(w * kWindow + 32 * t) * PITCH) = __builtin_bit_cast(tw_u32x2, v[t]);
        }
        const bool steps = active && s0 < s1;
        StepRegs<NC> rg;
        if (steps) prefetch_first_steps<NC, NCB>(rg, gt, bt, s0, s1, lane);
        if (j + 2 < n_loc) issue(j + 2);
        tw_lds_wait<63>();                                   // the chunk is there
        if (steps) run_steps<DT, MS, NC, NCB>(acc, rg, smem + half * 64, PITCH, gt, bt, s0, s1, lane);
        s0 = s1;
        s1 = fetch_int(sp, j + 2 <= n_loc ? j + 2 : n_loc);
        if (j + 1 < n_loc) tw_lds_wait<63>();                // everyone is done with it
    }
    if (active) {
        float* dst = p.partials + ((((long)part * p.n_mblocks + mb) * p.T + ti) * 2 + half) * (long)(NCB * 1024) + cg * (NC * 1024);
        if constexpr (H == 2) dump_partial<1, NC>(dst, acc, lane);
        else dump_partial<2, NC>(dst, acc, lane);
    }
}

}  // namespace

// ---- kernel tables
// The kernels can be compiled as eight translation units (-DTW_PART=1..4: fp16 / bf16 x plain / fused epilogue, 5..8:
// the same for TEW blobs) beside the host code (-DTW_PART=0), so that a build runs them in parallel; without TW_PART one unit holds
// everything.  The tables hand out host-side kernel addresses, so no type of this file crosses a unit boundary.
namespace tw_parts {
// (nta: the streamed kernels' variant whose requests for activations carry the streaming hint)
// (EW: the variant with the code of the element-wise residual, for TEW blobs)
template <int DT, bool FUSED, bool EW> const void* pick_mode(int mode, int ms, int ncb, bool nta);     // row-major boundary
template <int DT, bool FUSED, bool EW> const void* pick_mode_t(int mode, int ms, int ncb, bool nta);   // transposed boundary
template <int DT, bool FUSED> const void* pick_reduce(int ncb, bool transposed);               // second kernel of split K
template <int DT, bool FUSED> const void* pick_team(int ncb, bool transposed);                 // teams of waves per tile
template <int DT, bool FUSED> const void* pick_narrow(int ncb);                                // K resident, 64 rows, narrow staging windows
template <int DT> const void* pick_part(int ncb, int tiles);                                    // split K, row-major
template <int DT, bool FUSED> const void* pick_stream(int ncb);                     // K streamed, row-major
template <int DT, bool FUSED> const void* pick_rows(int ncb, int stages);                                  // a tile of a token block per workgroup
}  // namespace tw_parts

#if !defined(TW_PART) || TW_PART != 0
namespace {
template <int DT, int MS, int MODE, bool FUSED, bool TRANS, bool EW, bool NTA = true>
const void* pick_ncb(int ncb) {
    switch (ncb) {
        case 1: return (const void*)tw_gemm_kernel<DT, MS, 1, MODE, FUSED, TRANS, NTA, EW>;
        case 2: return (const void*)tw_gemm_kernel<DT, MS, 2, MODE, FUSED, TRANS, NTA, EW>;
        case 4: return (const void*)tw_gemm_kernel<DT, MS, 4, MODE, FUSED, TRANS, NTA, EW>;
        default: return nullptr;
    }
}
}  // namespace
namespace tw_parts {
template <int DT, bool FUSED, bool EW>
const void* pick_mode(int mode, int ms, int ncb, bool nta) {
    if (mode == 0) return ms == 2 ? pick_ncb<DT, 2, 0, FUSED, false, EW>(ncb) : pick_ncb<DT, 1, 0, FUSED, false, EW>(ncb);
    if (ms != 2) return nullptr;                  // the streamed kernels take 64-row blocks
    if (mode == 1) return nta ? pick_ncb<DT, 2, 1, FUSED, false, EW, true>(ncb) : pick_ncb<DT, 2, 1, FUSED, false, EW, false>(ncb);
    if (mode == 3) {                              // split K: the epilogue is the second kernel's, so only the plain variant exists
        if constexpr (!FUSED) return nta ? pick_ncb<DT, 2, 3, false, false, EW, true>(ncb) : pick_ncb<DT, 2, 3, false, false, EW, false>(ncb);
        else return nullptr;
    }
    return nta ? pick_ncb<DT, 2, 2, FUSED, false, EW, true>(ncb) : pick_ncb<DT, 2, 2, FUSED, false, EW, false>(ncb);
}
// transposed boundary: resident K with blocks of 64 or 32 tokens, streamed K always with 64
template <int DT, bool FUSED, bool EW>
const void* pick_mode_t(int mode, int ms, int ncb, bool nta) {
    if (mode == 0) return ms == 2 ? pick_ncb<DT, 2, 0, FUSED, true, EW>(ncb) : pick_ncb<DT, 1, 0, FUSED, true, EW>(ncb);
    if (ms != 2) return nullptr;
    if (mode == 1) return nta ? pick_ncb<DT, 2, 1, FUSED, true, EW, true>(ncb) : pick_ncb<DT, 2, 1, FUSED, true, EW, false>(ncb);
    if (mode == 3) {
        if constexpr (!FUSED) return nta ? pick_ncb<DT, 2, 3, false, true, EW, true>(ncb) : pick_ncb<DT, 2, 3, false, true, EW, false>(ncb);
        else return nullptr;
    }
    return nta ? pick_ncb<DT, 2, 2, FUSED, true, EW, true>(ncb) : pick_ncb<DT, 2, 2, FUSED, true, EW, false>(ncb);
}
template <int DT, bool FUSED>
const void* pick_reduce(int ncb, bool transposed) {
    switch (ncb) {
        case 1: return transposed ? (const void*)tw_splitk_reduce_kernel<DT, 1, FUSED, true> : (const void*)tw_splitk_reduce_kernel<DT, 1, FUSED, false>;
        case 2: return transposed ? (const void*)tw_splitk_reduce_kernel<DT, 2, FUSED, true> : (const void*)tw_splitk_reduce_kernel<DT, 2, FUSED, false>;
        case 4: return transposed ? (const void*)tw_splitk_reduce_kernel<DT, 4, FUSED, true> : (const void*)tw_splitk_reduce_kernel<DT, 4, FUSED, false>;
        default: return nullptr;
    }
}
template <int DT, bool FUSED>
const void* pick_narrow(int ncb) {
    switch (ncb) {
        case 1: return (const void*)tw_gemm_kernel<DT, 2, 1, 0, FUSED, false, true, false, kNarrowLines>;
        case 2: return (const void*)tw_gemm_kernel<DT, 2, 2, 0, FUSED, false, true, false, kNarrowLines>;
        case 4: return (const void*)tw_gemm_kernel<DT, 2, 4, 0, FUSED, false, true, false, kNarrowLines>;
        default: return nullptr;
    }
}
template <int DT>
const void* pick_part(int ncb, int tiles) {
    switch (ncb) {
        case 1: return tiles <= 4 ? (const void*)tw_part_kernel<DT, 1, 2, 1> : (const void*)tw_part_kernel<DT, 1, 1, 1>;
        case 2: return tiles <= 2 ? (const void*)tw_part_kernel<DT, 2, 2, 2> : tiles <= 4 ? (const void*)tw_part_kernel<DT, 2, 2, 1> : (const void*)tw_part_kernel<DT, 2, 1, 1>;
        case 4: return tiles <= 2 ? (const void*)tw_part_kernel<DT, 4, 2, 2> : tiles <= 4 ? (const void*)tw_part_kernel<DT, 4, 2, 1> : (const void*)tw_part_kernel<DT, 4, 1, 1>;
        default: return nullptr;
    }
}
template <int DT, bool FUSED>
const void* pick_stream(int ncb) {
    switch (ncb) {
        case 1: return (const void*)tw_stream_kernel<DT, 1, FUSED>;
        case 2: return (const void*)tw_stream_kernel<DT, 2, FUSED>;
        case 4: return (const void*)tw_stream_kernel<DT, 4, FUSED>;
        default: return nullptr;
    }
}
template <int DT, bool FUSED>
const void* pick_rows(int ncb, int stages) {
    switch (ncb) {
        case 1: return stages == 4 ? (const void*)tw_rows_kernel<DT, 1, FUSED, 4> : (const void*)tw_rows_kernel<DT, 1, FUSED, 8>;
        case 2: return stages == 4 ? (const void*)tw_rows_kernel<DT, 2, FUSED, 4> : (const void*)tw_rows_kernel<DT, 2, FUSED, 8>;
        case 4: return stages == 4 ? (const void*)tw_rows_kernel<DT, 4, FUSED, 4> : (const void*)tw_rows_kernel<DT, 4, FUSED, 8>;
        default: return nullptr;
    }
}
template <int DT, bool FUSED>
const void* pick_team(int ncb, bool transposed) {
    switch (ncb) {
        case 1: return transposed ? (const void*)tw_team_kernel<DT, 1, FUSED, true> : (const void*)tw_team_kernel<DT, 1, FUSED, false>;
        case 2: return transposed ? (const void*)tw_team_kernel<DT, 2, FUSED, true> : (const void*)tw_team_kernel<DT, 2, FUSED, false>;
        case 4: return transposed ? (const void*)tw_team_kernel<DT, 4, FUSED, true> : (const void*)tw_team_kernel<DT, 4, FUSED, false>;
        default: return nullptr;
    }
}
}  // namespace tw_parts
#endif

#ifdef TW_PART
#define TW_TABLES_EW(KW, DT, FUSED, EW)                                          \
    KW template const void* tw_parts::pick_mode<DT, FUSED, EW>(int, int, int, bool);  \
    KW template const void* tw_parts::pick_mode_t<DT, FUSED, EW>(int, int, int, bool);
#define TW_TABLES_REDUCE(KW, DT, FUSED)                                           \
    KW template const void* tw_parts::pick_reduce<DT, FUSED>(int, bool);          \
    KW template const void* tw_parts::pick_team<DT, FUSED>(int, bool);            \
    KW template const void* tw_parts::pick_rows<DT, FUSED>(int, int);            \
    KW template const void* tw_parts::pick_narrow<DT, FUSED>(int);                \
    KW template const void* tw_parts::pick_stream<DT, FUSED>(int);
#define TW_TABLES_ALL(KW, DT, FUSED) TW_TABLES_EW(KW, DT, FUSED, false) TW_TABLES_EW(KW, DT, FUSED, true) TW_TABLES_REDUCE(KW, DT, FUSED)
#define TW_TABLES_PART(KW, DT) KW template const void* tw_parts::pick_part<DT>(int, int);
#if TW_PART == 0
TW_TABLES_PART(extern, TW_F16) TW_TABLES_PART(extern, TW_BF16)
TW_TABLES_ALL(extern, TW_F16, false) TW_TABLES_ALL(extern, TW_F16, true) TW_TABLES_ALL(extern, TW_BF16, false) TW_TABLES_ALL(extern, TW_BF16, true)
#elif TW_PART == 1
TW_TABLES_EW(, TW_F16, false, false) TW_TABLES_REDUCE(, TW_F16, false) TW_TABLES_PART(, TW_F16)
#elif TW_PART == 2
TW_TABLES_EW(, TW_F16, true, false) TW_TABLES_REDUCE(, TW_F16, true)
#elif TW_PART == 3
TW_TABLES_EW(, TW_BF16, false, false) TW_TABLES_REDUCE(, TW_BF16, false) TW_TABLES_PART(, TW_BF16)
#elif TW_PART == 4
TW_TABLES_EW(, TW_BF16, true, false) TW_TABLES_REDUCE(, TW_BF16, true)
#elif TW_PART == 5
TW_TABLES_EW(, TW_F16, false, true)
#elif TW_PART == 6
TW_TABLES_EW(, TW_F16, true, true)
#elif TW_PART == 7
TW_TABLES_EW(, TW_BF16, false, true)
#elif TW_PART == 8
TW_TABLES_EW(, TW_BF16, true, true)
#else
#error "TW_PART is 0 (host code) or 1..8 (kernels)"
#endif
#endif

#if !defined(TW_PART) || TW_PART == 0
namespace {

// C[m, n] = act(bias[n]) (zero without a bias) for a weight with no surviving column.
template <int DT>
__global__ void tw_fill_kernel(unsigned short* C, long ldc, int M, int N, const unsigned short* bias, int act) {
    const long n = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long total = (long)M * N;
    for (long i = n; i < total; i += (long)gridDim.x * blockDim.x) {
        const long col = i % N;
        C[(i / N) * ldc + col] = bias ? tw_cvt<DT>(tw_activate(tw_to_f32<DT>(bias[col]), act)) : (unsigned short)0;
    }
}

// Ct[n, m] = act(bias[n]) (zero without a bias): the transposed output of a weight with no surviving column.
template <int DT>
__global__ void tw_fill_rows_kernel(unsigned short* Ct, long ldct, int N, int M, const unsigned short* bias, int act) {
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long total = (long)N * M;
    for (long i = t; i < total; i += (long)gridDim.x * blockDim.x) {
        const long n = i / M;
        Ct[n * ldct + (i % M)] = bias ? tw_cvt<DT>(tw_activate(tw_to_f32<DT>(bias[n]), act)) : (unsigned short)0;
    }
}

// ---- residual weights of a TEW blob in columns that keep no tile-wise weight (Sec. IV-A "Hybrid Pattern") ----
// The paper stores the element-wise part in CSC form and runs it as a sparse product of its own, added by
// linearity.  For the columns that own a packed column of a tile that happens inside the tiles' kernel; a
// column that the tile-wise pattern pruned altogether has none, so its few entries run here, after that
// kernel (which wrote the column's zeros, or act(bias)): C[m, n] = act(bias[n] + sum_e v_e * A[m, k_e]).
struct XcolParams {
    const unsigned short* A;
    unsigned short* C;
    const unsigned short* bias;
    const int* col;
    const int* ptr;
    const int* k;
    const unsigned short* v;
    const int* rank;            // position of a column among those of its tile
    long lda, ldc;
    int M, K, n_cols, act;
    int skip_below;             // columns with rank < skip_below were added by the tiles' kernel already
};

// Row-major boundary.  A workgroup takes 64 rows of A and 64 of the columns; wave w, lane r: row r, columns
// 16*w .. 16*w+15 of the group.  A comes through LDS in chunks of 256 K positions (coalesced 16-byte loads, the
// next chunk on its way in registers while this one is worked on), so that a lane's scattered 2-byte reads hit
// LDS, not memory; the entries of a column are walked in ascending K, chunk by chunk.  The wave holds 64 entries
// of each of its 16 columns, one entry per lane (fetched again when a column has used its 64 up), counts with a
// ballot how many of them lie inside the chunk and hands those round with v_readlane, four LDS reads in flight.
// (Fetched entry by entry, a column's 40 entries were 80 dependent round trips to memory: 220 us on the FFN-down
// of BERT-base against 60 now.)
constexpr int kXcChunk = 256, kXcPitch = 2 * kXcChunk + 8, kXcColsPerWg = 64;
template <int DT>
__global__ __launch_bounds__(256) void tw_xcol_kernel(const XcolParams p) {
    __shared__ __attribute__((aligned(16))) unsigned char at[64 * kXcPitch];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row0 = blockIdx.x * 64;
    const int j0 = blockIdx.y * kXcColsPerWg + 16 * wave;      // this wave's first column of the list
    float acc[16];
    int e[16], e1[16], base[16];                                // wave-uniform: next entry, end, entry that lane 0 holds
    int kreg[16];
    float vreg[16];
    auto fetch = [&](int i) {                                   // entries base[i] + lane of column i (clamped to its last)
        const int idx = base[i] + lane < e1[i] ? base[i] + lane : e1[i] - 1;
        const bool any = base[i] < e1[i];                        // wave-uniform
        kreg[i] = any ? p.k[idx] : 0x7fffffff;
        vreg[i] = any ? tw_to_f32<DT>(p.v[idx]) : 0.f;
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int j = j0 + i;
        acc[i] = 0.f;
        const bool mine = j < p.n_cols && p.rank[j] >= p.skip_below;
        e[i] = base[i] = __builtin_amdgcn_readfirstlane(mine ? p.ptr[j] : 0);
        e1[i] = __builtin_amdgcn_readfirstlane(mine ? p.ptr[j + 1] : 0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) fetch(i);
    const int kpad = (p.K + 7) & ~7;                             // rows are readable up to the next multiple of 8
    const unsigned char* arow = at + lane * kXcPitch;
    // staging of a chunk: 64 rows x 32 pieces of 16 bytes, eight per thread
    constexpr int kPieces = 64 * (kXcChunk / 8) / 256;
    tw_u32x4 stage[kPieces];
    auto request = [&](int c0) {
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const int id = tid + 256 * q;
            const int r = id / (kXcChunk / 8), pc = id % (kXcChunk / 8);
            int g = row0 + r;
            g = g < p.M ? g : p.M - 1;
            stage[q] = tw_u32x4{0u, 0u, 0u, 0u};
            if (c0 + 8 * pc < kpad) stage[q] = tw_load16_stream(p.A + (long)g * p.lda + c0 + 8 * pc);
        }
    };
    request(0);
    for (int c0 = 0; c0 < p.K; c0 += kXcChunk) {
        const int cend = c0 + kXcChunk;
        __syncthreads();                                         // everyone is through with the previous chunk
#pragma unroll
        for (int q = 0; q < kPieces; ++q) {
            const int id = tid + 256 * q;
            const int r = id / (kXcChunk / 8), pc = id % (kXcChunk / 8);
            *(tw_u32x2*)(at + r * kXcPitch + pc * 16) = tw_u32x2{stage[q].x, stage[q].y};
            *(tw_u32x2*)(at + r * kXcPitch + pc * 16 + 8) = tw_u32x2{stage[q].z, stage[q].w};
        }
        __syncthreads();
        if (cend < p.K) request(cend);                           // on its way while this chunk's entries are added
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            while (e[i] < e1[i]) {                               // (wave-uniform control flow)
                const int off = e[i] - base[i];                  // 0 .. 63: first unused entry among the 64 held
                const int held = e1[i] - base[i] < 64 ? e1[i] - base[i] : 64;
                // the held entries inside the chunk are consecutive from `off`: K ascends within a column
                const unsigned long long in = __builtin_amdgcn_ballot_w64(lane >= off && lane < held && kreg[i] < cend);
                const int n = __builtin_popcountll(in);
                auto a_of = [&](int t) {
                    const int k = __builtin_amdgcn_readlane(kreg[i], off + t);
                    return tw_to_f32<DT>(*(const unsigned short*)(arow + (k - c0) * 2));
                };
                auto w_of = [&](int t) {
                    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, vreg[i]), off + t));
                };
                int t = 0;
                for (; t + 4 <= n; t += 4) {
                    const float a0 = a_of(t), a1 = a_of(t + 1), a2 = a_of(t + 2), a3 = a_of(t + 3);
                    acc[i] += w_of(t) * a0;
                    acc[i] += w_of(t + 1) * a1;
                    acc[i] += w_of(t + 2) * a2;
                    acc[i] += w_of(t + 3) * a3;
                }
                for (; t < n; ++t) acc[i] += w_of(t) * a_of(t);
                e[i] += n;
                if (off + n < 64 || e[i] >= e1[i]) break;       // entries of a later chunk remain, or the column is done
                base[i] = e[i];                                  // all 64 used up: the column's next 64
                fetch(i);
            }
        }
    }
    const int m = row0 + lane;
    if (m < p.M) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int j = j0 + i;
            if (j < p.n_cols && p.rank[j] >= p.skip_below) {
                const int n = p.col[j];
                const float b = p.bias ? tw_to_f32<DT>(p.bias[n]) : 0.f;
                p.C[(long)m * p.ldc + n] = tw_cvt<DT>(tw_activate(acc[i] + b, p.act));
            }
        }
    }
}

// Transposed boundary: a column of C is a row of Ct and a K position a row of At, so a thread takes one token
// and the reads are coalesced as they are.  blockIdx.y walks the columns of the list.
template <int DT>
__global__ __launch_bounds__(256) void tw_xcol_t_kernel(const XcolParams p) {
    const long m = (long)blockIdx.x * 256 + threadIdx.x;
    if (m >= p.M) return;
    for (int j = blockIdx.y; j < p.n_cols; j += gridDim.y) {
        if (p.rank[j] < p.skip_below) continue;
        float acc = 0.f;
        int e = p.ptr[j];
        const int e1 = p.ptr[j + 1];
        // eight requests in flight per thread (one at a time, a column's 40 entries were 40 round trips to memory);
        // the products are added in the order of the entries either way
        for (; e + 8 <= e1; e += 8) {
            unsigned short a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = p.A[(long)p.k[e + u] * p.lda + m];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += tw_to_f32<DT>(p.v[e + u]) * tw_to_f32<DT>(a[u]);
        }
        for (; e < e1; ++e)
            acc += tw_to_f32<DT>(p.v[e]) * tw_to_f32<DT>(p.A[(long)p.k[e] * p.lda + m]);
        const int n = p.col[j];
        const float b = p.bias ? tw_to_f32<DT>(p.bias[n]) : 0.f;
        p.C[(long)n * p.ldc + m] = tw_cvt<DT>(tw_activate(acc + b, p.act));
    }
}

// Enqueues the pass over the residual's columns without tile-wise weights, if the blob has any.
int launch_xcols(const TwHeader* h, const void* blob_dev, const void* A, long lda, void* C, long ldc, int M,
                 const void* bias, int act, bool transposed, hipStream_t stream, bool inline_done = false) {
    if (h->xc_n <= 0 || M <= 0) return TW_OK;
    if (inline_done && h->xc_overflow == 0) return TW_OK;   // the tiles' kernel added them all
    const unsigned char* b = (const unsigned char*)blob_dev;
    XcolParams p;
    p.A = (const unsigned short*)A; p.C = (unsigned short*)C; p.bias = (const unsigned short*)bias;
    p.col = (const int*)(b + h->off_xc_col); p.ptr = (const int*)(b + h->off_xc_ptr);
    p.k = (const int*)(b + h->off_xc_k); p.v = (const unsigned short*)(b + h->off_xc_v);
    p.rank = (const int*)(b + h->off_xc_rank);
    p.lda = lda; p.ldc = ldc; p.M = M; p.K = h->K; p.n_cols = h->xc_n; p.act = act;
    p.skip_below = inline_done ? TW_XC_INLINE : 0;
    void* args[] = {(void*)&p};
    hipError_t rc;
    if (transposed) {
        const unsigned gy = (unsigned)(h->xc_n < 65535 ? h->xc_n : 65535);
        const void* fn = h->dtype == TW_F16 ? (const void*)tw_xcol_t_kernel<TW_F16> : (const void*)tw_xcol_t_kernel<TW_BF16>;
        rc = hipLaunchKernel(fn, dim3((unsigned)((M + 255) / 256), gy), dim3(256), args, 0, stream);
    } else {
        const long gy = ((long)h->xc_n + kXcColsPerWg - 1) / kXcColsPerWg;
        if (gy > 65535) return TW_ERR_UNSUPPORTED;
        const void* fn = h->dtype == TW_F16 ? (const void*)tw_xcol_kernel<TW_F16> : (const void*)tw_xcol_kernel<TW_BF16>;
        rc = hipLaunchKernel(fn, dim3((unsigned)((M + 63) / 64), (unsigned)gy), dim3(256), args, 0, stream);
    }
    return rc == hipSuccess ? TW_OK : TW_ERR_HIP;
}

struct Plan {
    int mode;       // kernel MODE
    int ms;         // the kernel's MS
    int n_mblocks, n_seg, n_items;
    int tiles_per_set;   // streamed K: tiles a workgroup holds
    int row_step;        // rows per row block (see TwGemmParams)
    unsigned at_pitch, abuf_bytes, stage_off, misc_off, lds_bytes;
    unsigned urow_off;   // transposed boundary, loading waves: LDS offset of their row lists (0: whole chunks are read)
    unsigned xbuf_off;   // row-major boundary, K resident, TEW blob with residual-only columns: LDS offset of the waves' areas for them
    int n_parts, chunks_per_part;   // split K (see TwGemmParams); n_parts = 1: none
    int team_shift;                 // log2 of the waves that share a tile (tw_team_kernel), 0: none
    int rows_group;                 // tw_rows_kernel: token blocks walked together, 0: another kernel runs
    int rows_stages;                // and the depth of its ring
    unsigned rows_lds;              // and its on-chip memory per workgroup
    bool narrow;                    // K resident, 64 rows: narrow staging windows
    int stream_items;               // tw_stream_kernel: its items, 0: another kernel runs
    size_t partial_bytes;           // workspace the parts' fp32 results take, behind the counters
};


constexpr unsigned kLdsLimit = 160 * 1024;
// Estimates of the planner for streamed K when a launch has fewer items than compute units, in microseconds
// (fitted to the FFN-down of BERT-base and of BERT-large and to a lowered convolution, K = 2304 .. 4096 in 6 to 11
// chunks, M = 64 .. 6000, both boundaries).  Unsplit: kItemUs for the launch and the start of an item, then per
// chunk in sequence kChunkUs (what it takes a compute unit to bring in 64 rows x 384 columns of A; kChunkUsT on
// the transposed boundary, where whole rows go to LDS; kNarrowChunk of it for tiles of at most 64 columns, whose
// requests run two chunks ahead).  Split: kSplitItemUs (nothing overlaps the first chunk), a chunk takes longer
// the more workgroups stream at once (1 + kLoadedChunk at a full round), the tiles' partial results leave a
// compute unit at kCuStoreBytesPerUs; the second kernel costs kReduceUs plus, per wave that a compute unit gets,
// kReduceWaveUs and its loads at kCuLoadBytesPerUs.  A split must promise kSplitMargin of the unsplit time or less.
// (The constants are older than the second kernel's requests ahead: of 91 split plans timed, the estimate is 1.3 times the
// measured time in the median, and the split is 1.08 to 4 times as fast as the same call unsplit.  It errs to the unsplit side.)
constexpr double kItemUs = 4.5, kChunkUs = 3.3, kChunkUsT = 2.8, kNarrowChunk = 0.85, kSplitItemUs = 5.5,
                 kLoadedChunk = 0.4, kCuStoreBytesPerUs = 38e3, kReduceUs = 2.5, kReduceWaveUs = 0.25,
                 kCuLoadBytesPerUs = 24e3, kSplitMargin = 0.9;

unsigned at_bytes(int msb, int k_chunk) {
    const unsigned pitch = 64u * msb + 8u;
    return ((unsigned)(k_chunk + 9) * pitch + 15u) & ~15u;
}
unsigned lds_need(int msb, int k_chunk, int buffers) {
    return buffers * at_bytes(msb, k_chunk) + kWaves * kStageBytes + 16u;
}
// Most steps that a tile has.  The tiles are ordered by kept rows; with several chunks each chunk's rows are rounded up to whole steps,
// so a tile whose rows are spread can have more steps than one that keeps more of them (20 rows in 12 chunks: 12 steps; 21 in
// one chunk: 2).
int heaviest_steps(const TwHeader* h) {
    const unsigned char* blob = (const unsigned char*)h;
    const TwTileDesc* d = (const TwTileDesc*)(blob + h->off_tile_desc);
    int most = d[*(const int32_t*)(blob + h->off_sched_order)].nsteps;
    for (int t = 0; h->n_chunks > 1 && t < h->T; ++t) most = d[t].nsteps > most ? d[t].nsteps : most;
    return most;
}
// 64 rows of a resident K beside narrow staging windows
unsigned lds_need_narrow(int k) { return at_bytes(2, k) + kWaves * kNarrowStageBytes + 16u; }

// Estimate of an item with K resident, in microseconds: launch and first operands, bringing in 32 * msb rows of A while the
// whole chip does, and then whichever takes longer: the packed weights of its tiles through the compute unit's vector L1
// and the stores; or a wave's tiles one after the other, each with the steps of a heavy tile (half again as many as the
// mean) and an epilogue, which GELU lengthens.  It serves to compare the plans of one call.  On 640 calls (64 to 900 columns of
// A, 700 to 8192 rows) timed with 32-row and with 64-row blocks in one round, its choice takes 0.8 % more than the faster one
// on average, more than a tenth in 2 % of them; without the epilogue in the chain it was 2.3 % and 7 % (320 -> 3381, G =
// 32, GELU, at 989 rows: 13.6 us with 64-row blocks and seven tiles for eight waves, 15.5 with 32 rows and thirteen).  What it
// does not see is a heavy tile among many light ones: 256 -> 3008 at 4096 tokens, transposed, takes 12.6 us by it, 10.9 with 64 rows.
// kRoundMargin: with K > kMarginK one round of workgroups is left for several only for a tenth of its time (a second round
// brings all of A in again, at more than the estimate has for it).  Of 128 calls whose best estimate is a second round 1 to
// 9 % below one round, one round was the faster by 14 % on average (0.90 to 1.42 times; 1065 -> 1927 at 5370 rows 1.2); TEW blobs
// alike.  Of 64 such calls with shorter K the second round was the faster by 2 % (0.85 to 1.17), of TEW blobs by 12 %: 678 ->
// 2304 (G = 32) at 8338 rows 76 us, 85 in one round.  Between two rounds and more the estimate needs no margin: the items
// are then pulled as they come and more of them even out, so plans that it puts 0.1 to 10 % lower took 0.86 to 1.02
// times as long row-major, 0.88 to 1.06 transposed.
constexpr double kRoundMargin = 0.9;
constexpr int kMarginK = 768;

double resident_item_us(const TwHeader* h, int msb, int tiles, int team_shift, bool gelu) {
    constexpr double kStartUs = 5.0, kStageBytesPerUs = 20e3, kWeightBytesPerUs = 70e3, kStoreBytesPerUs = 32e3, kStepUs = 0.1,
                     kEpilogueUs = 1.5, kGeluUs = 2.0, kTallEpilogue = 1.4;
    const double steps = (double)h->total_steps / h->T;
    const double through = tiles * (steps * h->ncb * 1024.0 / kWeightBytesPerUs + 64.0 * msb * h->G / kStoreBytesPerUs);
    const double epilogue = (kEpilogueUs + (gelu ? kGeluUs * h->G / 128.0 : 0.0)) * (msb > 1 ? kTallEpilogue : 1.0);
    const double chain = ((tiles + kWaves - 1) / kWaves) * (1.5 * steps * kStepUs / (1 << team_shift) + epilogue);
    return kStartUs + 64.0 * msb * h->K / kStageBytesPerUs + (through > chain ? through : chain);
}

// K resident, 32-row blocks, one round of workgroups with at most four tiles each: teams of waves may share the tiles
// (tw_team_kernel).  log2 of the waves to a tile, 0: a wave per tile.
// A team takes the heaviest tile's steps side by side and shares the epilogue out, and pays for it with the waves' sums
// through LDS.  What that saves and costs, in microseconds, was measured against a wave per tile on the same plans (2400
// calls, K = 48 .. 1536, 1 to 8000 rows, both boundaries, plain / bias / GELU): kTeamStepUs for every step of the heaviest tile and
// kTeamGeluUs for a shared GELU, against kTeamUs, more for two waves to a tile (they save the least) and with K > 768 (A then
// comes in in larger batches, which a wave per tile does for every K).  Teams taken by this line or always, the calls are 1.15
// us faster on average (1.18 with the faster kernel each time), but always taken some lose 1.6 us, by the line 0.9.
// 168 -> 3699 (G = 128) at 934 rows 9.8 us with a wave per tile, 10.6 with teams; 768 -> 768 (G = 128) at 256 rows 9.9 and 7.7.
// The choice decides in which groups a result's products are summed, so it must not depend on the boundary nor on a bias
// or ReLU: both boundaries give the same bits, and so do a fused and a separate ReLU.
int team_of(const TwHeader* h, int msb, int most_tiles, long items, int n_cu, bool gelu) {
    if (msb != 1 || items > n_cu || most_tiles > kWaves / 2 || h->ew_nnz > 0) return 0;
    constexpr double kTeamStepUs[3] = {0.046, 0.055, 0.085};          // tiles of 1, 2, 4 column blocks
    constexpr double kTeamUs[3] = {-0.1, 0.0, 0.2}, kTwoWavesUs[3] = {0.0, 0.1, 0.5}, kLongUs[3] = {0.3, 0.7, 0.5},
                     kTeamGeluUs[3] = {0.5, 0.8, 1.4};
    const int shift = most_tiles <= 1 ? 3 : most_tiles <= 2 ? 2 : 1;
    const int width = h->ncb >= 4 ? 2 : h->ncb - 1;
    double cost = kTeamUs[width];
    if (shift == 1) cost += kTwoWavesUs[width];
    if (h->K > 768) cost += kLongUs[width] + (shift == 1 && width == 2 ? 0.9 : 0.0);
    if (gelu) cost -= kTeamGeluUs[width];
    return kTeamStepUs[width] * heaviest_steps(h) > cost ? shift : 0;
}

int make_plan(const TwHeader* h, int M, int n_cu, Plan& pl, bool transposed = false, size_t ws_avail = ~(size_t)0,
              bool gelu = false, bool narrow_windows = true) {
    const bool resident = h->n_chunks == 1;
    const int buffers = resident ? 1 : 2;
    if (lds_need(1, h->k_chunk, buffers) > kLdsLimit) return TW_ERR_UNSUPPORTED;
    const int T = h->T;
    // msb: 32-row blocks in a workgroup's row block; tpw: tiles a workgroup of the streamed kernel holds
    int segs = 1;                // resident K: workgroups that share a row block's tiles
    auto items_for = [&](int msb, int tpw, int& n_mblocks, int& n_seg) {
        n_mblocks = (M + 32 * msb - 1) / (32 * msb);
        n_seg = resident ? segs : (T + tpw - 1) / tpw;
        return (long)n_mblocks * n_seg;
    };
    int msb = 2, tpw = kWaves;
    int nmb, nseg;
    // 64 rows with narrow staging windows (K from 921 to 1040; the row-major boundary's plain blobs): the packed weights of 64 rows are
    // streamed once instead of twice.  Not where the heaviest tile has more than kSkew times the mean's steps: it is one wave's, with
    // 64 rows twice as long (3025 x 1024 -> 1167, skewed, 22.3 us, 19.4 in 32 rows; 8192 x 1024 -> 4096, skewed, 2 % slower), and only for
    // kNarrowCost less of the estimate, which does not see a wide tile's second window (which is all there is to few wide tiles of few
    // steps: 49920 x 1035 -> 832, 8 steps a tile, 75.4 us, 72.2 in 32 rows).
    constexpr double kSkew = 2.5, kNarrowCost = 1.06;
    const bool narrow = narrow_windows && resident && !transposed && h->ew_nnz == 0 && lds_need(2, h->k_chunk, 1) > kLdsLimit && lds_need_narrow(h->k_chunk) <= kLdsLimit &&
                        (double)heaviest_steps(h) * T <= kSkew * (double)h->total_steps && (h->ncb < 4 || T > kWaves || h->total_steps >= 12L * T);
    if (lds_need(2, h->k_chunk, buffers) > kLdsLimit && !narrow) msb = 1;
    pl.mode = resident ? 0 : 1;
    if (resident) {
        // 64-row blocks with all tiles when they give every compute unit an item.  With fewer the height of the row blocks
        // and the workgroups per row block are what the estimate below finds fastest.  What it has to get right is
        // the number of rounds: a second one costs as much as the first, nothing of it overlaps.  (Before, the tiles
        // were shared out over ceil(units / row blocks) workgroups, which is up to twice as many as a round holds.)
        // Back to back in a graph, before ->
        // now: 768 -> 3072 at 1000 / 3000 / 12000 rows 13.1 -> 10.1, 34.5 -> 18.4, 54 -> 39.5 us; 768 -> 768 at 8192 15.8 -> 12.9;
        // 1400 -> 2000 at 3000 37 -> 20; 1000 -> 1234 (G = 32) at 4321 36.5 -> 25.3; transposed 768 -> 2304 at 6000 tokens
        // 35 -> 19.6, 500 -> 4000 (G = 32) at 5000 39 -> 23.0; 768 -> 3072 at 16384 and 17000 as before.
        const long nmb_full = (M + 32L * msb - 1) / (32 * msb);
        if (nmb_full < n_cu || msb == 1 || narrow) {
            // (only shares that give a workgroup fewer tiles than the one before: about 2 sqrt(T) of them)
            double best = 0.0, one_round = 0.0;
            int one_msb = msb, one_segs = 1;
            for (int m = M <= 32 ? 1 : msb; m >= 1; --m) {
                const long blocks = (M + 32L * m - 1) / (32 * m);
                // (sharing a row block's tiles out any further than this only adds rounds)
                const long most_segs = blocks < n_cu ? 2 * n_cu / blocks + 1 : 3;
                for (int sg = 1; sg <= most_segs;) {
                    const int tiles = (T + sg - 1) / sg;
                    const long rounds = (blocks * sg + n_cu - 1) / n_cu;
                    const double cost = (narrow && m == 2 ? kNarrowCost : 1.0) * rounds * resident_item_us(h, m, tiles, team_of(h, m, tiles, blocks * sg, n_cu, gelu), gelu);
                    if (best == 0.0 || cost < best) { best = cost; msb = m; segs = sg; }
                    if (rounds == 1 && (one_round == 0.0 || cost < one_round)) { one_round = cost; one_msb = m; one_segs = sg; }
                    if (tiles == 1) break;
                    sg = (T + tiles - 2) / (tiles - 1);
                }
            }
            if (one_round > 0.0 && best > kRoundMargin * one_round && h->K > kMarginK) { msb = one_msb; segs = one_segs; }
            // in one round: a tile fewer for as many workgroups as there is room for
            const long blocks = (M + 32L * msb - 1) / (32 * msb);
            if (blocks * segs <= n_cu) segs = (int)(n_cu / blocks < T ? n_cu / blocks : T);
        }
    } else if (msb == 2) {
        // Streamed K, 64-row blocks.  Eight tiles per workgroup (a wave per tile) when that gives every compute
        // unit an item and there are more than four tiles.  Else four waves multiply and four only load A
        // (MODE 2), with as many tiles per workgroup (4, 2, 1) as still fill the GPU: fewer tiles per workgroup
        // mean more workgroups per row block, each reading the block's rows of A again (from the caches).
        // Measured: skewed FFN-down of BERT-large, M = 8192, T = 8: 45 us with sets of four against 57 us with
        // 32-row blocks and a wave per tile; FFN-down of BERT-base, M = 512: see the design notes.
        if (T <= kWaves / 2 || items_for(2, kWaves, nmb, nseg) < n_cu) {
            pl.mode = 2;
            tpw = kWaves / 2;
            while (tpw > 1 && items_for(2, tpw, nmb, nseg) < n_cu) tpw >>= 1;
            // (an item takes about as long with fewer tiles, its time is the time to bring A in: one round of
            // workgroups that leaves compute units idle beats two rounds)
            if (tpw < kWaves / 2 && items_for(2, tpw, nmb, nseg) > n_cu) tpw <<= 1;
        }
    }
    if (!resident && msb != 2) return TW_ERR_UNSUPPORTED;   // (the streamed kernels take 64-row blocks; 384-row chunks fit)
    pl.ms = msb;
    long items = items_for(msb, tpw, nmb, nseg);
    if (items > 0x7fffffffL) return TW_ERR_UNSUPPORTED;
    pl.row_step = 32 * msb;
    // Row-major boundary, two to four rounds of 64-row blocks, the last one partly empty (M = 20001: 313 blocks
    // on 256 compute units): lower row blocks fill the last round, and every block then brings in and stores
    // fewer rows (40 instead of 64: 86 us instead of 100 us on the FFN-up of BERT-base).  With more rounds the
    // empty part of the last one weighs little and the extra blocks cost as much as they gain (the conv
    // workload, 6.1 rounds: no change with 56-row blocks).  The transposed boundary keeps 64 tokens: a block's
    // tokens are whole 128-byte lines of the output there.
    if (!transposed && msb == 2 && items > n_cu && items <= 4L * n_cu && items % n_cu != 0) {
        const long rounds = (items + n_cu - 1) / n_cu;
        const long blocks = rounds * n_cu / nseg;                 // row blocks that fit into that many rounds
        int rows = (int)(((M + blocks - 1) / blocks + 7) / 8 * 8);
        if (rows > 32 && rows < 64) {
            pl.row_step = rows;
            nmb = (M + rows - 1) / rows;
            items = (long)nmb * nseg;
        }
    }
    if (!resident && 4 * msb * ((((h->k_chunk + 7) >> 3) + 7) >> 3) > kWaves * 6) return TW_ERR_UNSUPPORTED;   // a chunk is one batch
    pl.n_mblocks = nmb; pl.n_seg = nseg; pl.n_items = (int)items;
    pl.at_pitch = 64u * msb + 8u;
    pl.abuf_bytes = at_bytes(msb, h->k_chunk);
    pl.stage_off = buffers * pl.abuf_bytes;
    pl.narrow = narrow && msb == 2;
    pl.misc_off = pl.stage_off + kWaves * (pl.narrow ? kNarrowStageBytes : kStageBytes);
    pl.lds_bytes = pl.misc_off + 16u;
    pl.tiles_per_set = resident ? 0 : tpw;
    // Transposed boundary, at most four tiles, streamed: the loading waves read only the K rows the tiles keep,
    // from lists they hold in LDS.  (The blob's row lists are per set of TW_SET_TILES(T) tiles: with other sets
    // the loading waves bring in whole chunks.)
    pl.urow_off = 0;
    if (transposed && pl.mode == 2 && T <= kWaves / 2 && tpw == kWaves / 2) {
        const unsigned need = (kWaves / 2) * (unsigned)h->n_chunks * (8 * 12 + 2) * 2;
        if (pl.lds_bytes + need <= kLdsLimit) { pl.urow_off = pl.lds_bytes; pl.lds_bytes += need; }
    }
    // per-wave areas for the residual-only columns that the tiles add themselves (TEW), if there is room left
    pl.xbuf_off = 0;
    if (h->xc_n > 0) {
        const unsigned need = kWaves * TW_XC_INLINE * 64 * 2;
        if (pl.lds_bytes + need <= kLdsLimit) { pl.xbuf_off = pl.lds_bytes; pl.lds_bytes += need; }
    }
    // Split K.  With streamed K and few row blocks the plan above leaves most compute units idle while each
    // workgroup walks all chunks in sequence, and a compute unit brings A in at about 16 KB per microsecond only
    // (its queue of outstanding misses times the memory latency), 3 us per chunk.  The alternative: MODE 1 with
    // the chunks cut into parts of equal length and the tiles into sets of `tpw`, an item per (part, set, row
    // block), all in one round; the tiles' fp32 results go to the workspace and a second kernel adds them in a
    // fixed order and stores C.  Both the number of parts and the tiles per set are chosen by the estimate below;
    // the split is taken when its estimate is lower and the caller's workspace holds the partial results.
    // (Not where the tiles add the residual-only columns of a TEW blob themselves: a split leaves those to the pass
    // of their own, which reads all of A once more - 92 against 46 us on the FFN-down of BERT-base at 512 rows.)
    pl.n_parts = 1; pl.chunks_per_part = h->n_chunks; pl.partial_bytes = 0;
    // Teams of waves (see team_of).  Calls back to back in a graph, a wave per tile -> teams: 768 -> 3072 at 1 / 64 / 512 rows
    // 8.2 / 9.9 / 10.3 -> 7.5 / 8.5 / 8.9 us, 768 -> 768 at 256 / 2048 rows 9.9 / 10.7 -> 8.5 / 8.9 us, transposed
    // 768 -> 2304 at 512 tokens 8.2 -> 7.0 us, 1500 -> 800 at 100 tokens 11.5 -> 8.0 us.  With five tiles or more nearly every
    // wave has a tile of its own.  (TEW blobs stay with a wave per tile: a tile's residual has steps of another kind.)
    pl.team_shift = resident ? team_of(h, msb, (T + nseg - 1) / nseg, items, n_cu, gelu) : 0;
    if (pl.team_shift > 0) {
        const unsigned sums = (unsigned)kWaves * h->ncb * 4096u;      // the waves' fp32 sums, over A and the staging areas
        if (sums > pl.lds_bytes) pl.lds_bytes = sums;
    }
    if (!resident && msb == 2 && h->n_chunks >= 2 && (pl.xbuf_off == 0 || transposed)) {
        const long nmb1 = (M + 63) / 64;
        const size_t tile_bytes = (size_t)2 * h->ncb * 4096;          // fp32 results of a tile: 64 rows x G columns
        const int sub = transposed ? h->ncb : 8;                      // pieces of a tile in the second kernel
        const long units2 = nmb1 * T * sub;
        const double rounds0 = (double)((items + n_cu - 1) / n_cu);
        const double chunk_us = transposed ? kChunkUsT : kChunkUs;
        double best = rounds0 * (kItemUs + h->n_chunks * chunk_us * (h->ncb <= 2 ? kNarrowChunk : 1.0));
        int best_cpp = 0, best_tpw = 0;
        for (int sets = 1; sets <= T && nmb1 * sets * 2 <= n_cu; ++sets) {   // (at least two parts in one round)
            const int tpw1 = (T + sets - 1) / sets;
            if (tpw1 > kWaves || (sets > 1 && (T + sets - 2) / (sets - 1) == tpw1)) continue;   // (as many tiles per set with fewer sets)
            for (int cpp = h->n_chunks - 1; cpp >= 1; --cpp) {
                const int parts = (h->n_chunks + cpp - 1) / cpp;
                if (nmb1 * sets * parts > n_cu) break;
                if (cpp > 1 && (h->n_chunks + cpp - 2) / (cpp - 1) == parts) continue;   // a shorter part with as many parts follows
                const size_t bytes = (size_t)parts * nmb1 * T * tile_bytes;
                if (256 + bytes > ws_avail) continue;
                const double waves2 = (double)((units2 + n_cu - 1) / n_cu);     // of the second kernel, per compute unit
                const double loaded = 1.0 + kLoadedChunk * (double)(nmb1 * sets * parts) / n_cu;
                const double cost = kSplitItemUs + cpp * chunk_us * loaded + tpw1 * (double)tile_bytes / kCuStoreBytesPerUs +
                                    kReduceUs + waves2 * (kReduceWaveUs + parts * (double)(tile_bytes / sub) / kCuLoadBytesPerUs);
                if (cost < kSplitMargin * best) { best = cost / kSplitMargin; best_cpp = cpp; best_tpw = tpw1; }
            }
        }
        if (best_cpp > 0) {
            pl.mode = 1; pl.tiles_per_set = best_tpw; pl.row_step = 64; pl.urow_off = 0; pl.xbuf_off = 0;
            pl.chunks_per_part = best_cpp;
            pl.n_parts = (h->n_chunks + best_cpp - 1) / best_cpp;
            pl.n_mblocks = (int)nmb1; pl.n_seg = (T + best_tpw - 1) / best_tpw;
            pl.n_items = (int)(nmb1 * pl.n_seg * pl.n_parts);
            pl.partial_bytes = (size_t)pl.n_parts * nmb1 * T * tile_bytes;
            pl.lds_bytes = pl.misc_off + 16u;
        }
    }
    // What the narrow windows save is a round of workgroups.  Of 2809 random calls of such a K (1000 rows and more) that would take them, timed
    // both ways, 2101 take fewer rounds with them, 1.23 times as fast, 47 slower by more than 2 %.  Not among these: wide tiles in two rounds
    // instead of three (69 of 101 slower, 4 % on average: a wide tile has a second window).  And in one round either way 32 rows are ahead
    // unless a wave has its fourth tile there: 204 of 286 calls slower by 64 rows, 8 % on average (2832 x 1027 -> 1522, G = 128, 18.8 us in 32
    // rows, 27.5 in 64; 1693 x 1013 -> 3997 27 and 38); with more tiles 64 rows are 1.16 times as fast, 8 of 221 slower.
    // Nor where 32 rows have teams of waves: these sum in other groups, and the transposed boundary, which has no such windows, would have them.
    if (pl.narrow) {
        Plan low;
        if (make_plan(h, M, n_cu, low, transposed, ws_avail, gelu, false) != TW_OK) return TW_OK;
        const int rounds = (pl.n_items + n_cu - 1) / n_cu, low_rounds = (low.n_items + n_cu - 1) / n_cu;
        const int low_tiles = (T + low.n_seg - 1) / low.n_seg;
        if (low.team_shift > 0 || (low_rounds == 1 && low_tiles <= 3 * kWaves) || (h->ncb == 4 && rounds == 2 && low_rounds == 3)) pl = low;
    }
    return TW_OK;
}

// Whether tw_gemm_t runs tw_rows_kernel instead of the plan's kernel (pl.rows_group, 0: no).
// Not for plans that share a tile's K steps out (split K, teams of waves: other groups of sums), not for TEW blobs.  Otherwise
// the workgroups of that kernel are many and short, and it is the faster one wherever two things take less time than the plan's
// kernel as a whole: its longest workgroup (kRowsUs and kRowsStepUs for each step of the heaviest tile, kRowsCrowdUs with four workgroups to
// a compute unit, kRowsFar times that where fewer than eight token blocks leave the rows of all of them to every XCD and its L2 does not
// hold them), and what a compute unit puts through with all its workgroups (kRowsFullStepUs a step, 8 to 10 KB of rows and weights whatever the
// tile's width, and the stores).  The second decides on many narrow tiles: 16384 tokens of 768 -> 3072 (75 %) with G = 32 take 57 us here and 46 with
// the block of 64 tokens resident, with G = 64 43 and 43, with G = 128 39 and 44.  The plan's estimate, made to compare plans, is corrected by kPlan:
// its measured time is 0.68 to 0.88 of it with tiles of 32 columns, 1.06 to 1.17 resident with 128.
// Three kinds of calls keep the plan's kernel whatever the estimates, which do not see what is different there.  18300 random calls (16 to 200000
// tokens, K = 64 .. 6000, all widths and skews, plain and fused) were timed both ways; of those that the estimates would take this kernel is the slower one in:
// - one block of tokens, tiles of 64 columns, K resident: 17 of 23 (no load on the memory, the plan's kernel takes 5.4 to 6.5 us; 64 tokens of
//   896 -> 1979 6.0 us, 7.4 here);
// - tiles of 64 columns, K streamed in one round, a tile of more than 100 steps, at most 32 blocks: 70 of 104 (the wave that has the tile takes 0.14 us a step,
//   a workgroup of this kernel's two to a compute unit 0.17; 2266 tokens of 5120 -> 704 47 us, 60 here);
// - at most eight tiles of 32 columns, K streamed in full rounds, a tile of more than 180 steps: 41 of 47 (a compute unit holds two such lists,
//   and every tile's rows come from memory again; 42298 tokens of 5760 -> 120 154 us, 232 here).
// Of the 18300 calls this kernel is taken 15600 times, 1.61 times as fast in the geometric mean; 177 are slower than the plan's kernel by more than 2 %, 108 by
// more than 5 %, 44 by more than 10 % (most of them 32 or 64 columns, K streamed, tiles of 150 steps and more; without those lines and with the
// deeper ring for short tiles 419, 282 and 140).
void plan_rows(const TwHeader* h, int M, long lda, int n_cu, Plan& pl, bool gelu) {
    constexpr double kRowsUs = 6.5, kRowsStepUs = 0.14, kRowsCrowdUs = 0.18, kRowsGeluUs = 2.0, kTileStepUs = 0.15,
                     kRowsFullUs = 4.0, kRowsFullStepUs = 0.105, kRowsStoreBytesPerUs = 18e3, kRowsFar = 1.35,
                     kWeightBytesPerUs = 110e3;
    constexpr long kRowsL2 = 3400 * 1024;                    // of an XCD's 4 MiB, for rows of At
    constexpr int kDeepSteps = 24, kLongTile64 = 100, kLongTile32 = 180;
    pl.rows_group = 0;
    if (pl.n_parts > 1 || pl.team_shift > 0 || h->ew_nnz > 0 || h->n_chunks > 64) return;
    // (offsets below kRowsRange, products of 24-bit factors: from 1 GiB of At on the plan's kernel runs, whatever the estimates)
    if ((unsigned long)h->K * (unsigned long)lda * 2 >= kRowsRange || lda >= (1 << 23) || h->K >= (1 << 24)) return;
    const int heaviest = heaviest_steps(h);
    const int bt = h->ncb == 4 ? rows_bt<4>() : rows_bt<1>();
    const long blocks = ((long)M + bt - 1) / bt, items = blocks * h->T;
    if (items >= (1L << 24)) return;                         // (a launch holds 2^32 threads)
    const long rounds = ((long)pl.n_items + n_cu - 1) / n_cu;
    if (h->ncb == 2 && (h->n_chunks == 1 ? blocks == 1 : rounds == 1 && heaviest > kLongTile64 && blocks <= 32)) return;
    if (h->ncb == 1 && h->n_chunks > 1 && heaviest > kLongTile32 && h->T <= 8 && 10L * pl.n_items > 7 * rounds * n_cu) return;
    // two workgroups or fewer to a compute unit: a deeper ring takes the place of the others.  (Where two such rings do not fit beside each
    // other, tiles of 64 columns or long lists, one or fewer: a second round of workgroups costs as much as the first.  Not for tiles of
    // kDeepSteps or fewer, which end before it pays: in 4200 such calls the ring of four is 7 % faster in the median;
    // with 25 to 64 steps 4 %, but up to 3 % slower in a tenth of them, and above 64 the deeper ring is the faster one.)
    const unsigned stage = h->ncb == 4 ? rows_stage_bytes<4>() : h->ncb == 2 ? rows_stage_bytes<2>() : rows_stage_bytes<1>();
    auto lds_of = [&](int stages) { return stages * stage + (unsigned)(heaviest + stages + 1) * 64u; };
    pl.rows_stages = heaviest > kDeepSteps && items <= (2 * lds_of(8) <= kLdsLimit ? 2L : 1L) * n_cu ? 8 : 4;
    pl.rows_lds = lds_of(pl.rows_stages);
    if (pl.rows_lds > (pl.rows_stages == 8 ? kLdsLimit : 64u * 1024u)) return;
    // (a chunk's packed weights pass behind its rows of A: 590 steps, 22 us, of the 47.6 that 16384 tokens of 3072 -> 768 take there, 41.5 here)
    const double weights_us = (double)h->total_steps / pl.n_seg * h->ncb * 1024.0 / kWeightBytesPerUs;
    const double chunks_us = h->n_chunks * kChunkUsT * (h->ncb <= 2 ? kNarrowChunk : 1.0) + weights_us, tile_us = heaviest * (h->ncb <= 2 ? kTileStepUs : 1.5 * kTileStepUs);
    const double plan_us = rounds * (h->n_chunks == 1 ? resident_item_us(h, pl.ms, (h->T + pl.n_seg - 1) / pl.n_seg, 0, gelu)
                                                      : kItemUs + (chunks_us > tile_us ? chunks_us : tile_us));   // (a tile is one wave's there)
    const long bytes = (long)h->K * bt * 2;
    const double far = blocks < 8 && blocks * bytes > kRowsL2 ? kRowsFar : 1.0;
    const double longest_us = kRowsUs + heaviest * far * (pl.rows_stages == 8 ? kRowsStepUs : kRowsCrowdUs) + (gelu && items < n_cu ? kRowsGeluUs : 0.0);
    const double full_us = kRowsFullUs + ((double)blocks * h->total_steps * kRowsFullStepUs + (double)M * h->T * h->G * 2.0 / kRowsStoreBytesPerUs) / n_cu;
    const double kPlan = h->ncb == 1 ? (h->n_chunks > 1 ? 0.8 : pl.ms > 1 ? 0.77 : 0.75) : h->ncb == 4 && h->n_chunks == 1 ? 1.15 : 1.0;
    if ((longest_us > full_us ? longest_us : full_us) >= kPlan * plan_us) return;
    const long group = 8 * (bytes < kRowsL2 ? kRowsL2 / bytes : 1);
    pl.rows_group = (int)(group < blocks ? group : blocks < 8 ? 8 : blocks & ~7L);
}

// Whether tw_gemm runs tw_stream_kernel instead of the plan's kernel (pl.stream_items): wherever the plan is MODE 2, but for TEW blobs
// and pitches whose rows lie too far apart for 32-bit offsets.  (5400 random calls: 1.25 times as fast on average, see there.)
constexpr long kFarPitch = 1 << 23;
unsigned stream_lds_bytes() { return 2 * at_bytes(2, kStreamChunk) + kStreamTiles * kStageBytes + kWindows * kWindowBytes; }
void plan_stream(const TwHeader* h, long lda, Plan& pl) {
    pl.stream_items = 0;
    if (pl.mode != 2 || pl.n_parts > 1 || h->k_chunk != kStreamChunk || h->ew_nnz > 0 || lda >= kFarPitch) return;
    pl.stream_items = pl.n_items;
}

// Whether tw_gemm runs tw_part_kernel for a split's parts: for every split, but for TEW blobs (their residual's steps are in MODE 3) and those
// pitches.  (Of 4990 random split calls two are slower than with MODE 3 by more than 2 %, 1.23 times as fast on average.)
bool parts_by_direct_loads(const TwHeader* h, long lda, const Plan& pl) {
    return pl.n_parts > 1 && h->ew_nnz == 0 && h->k_chunk == kStreamChunk && lda < kFarPitch;
}
unsigned part_lds_bytes() { return at_bytes(2, kStreamChunk) + 2 * 64 * kStreamChunk * 2; }

// the kernel for (dtype, mode, MS, NCB, fused epilogue): a host-side address for hipLaunchKernel and hipFuncSetAttribute
template <bool EW>
const void* pick_kernel_t_of(int dt, int mode, int ms, int ncb, bool fused, bool nta) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_mode_t<TW_F16, true, EW>(mode, ms, ncb, nta) : pick_mode_t<TW_BF16, true, EW>(mode, ms, ncb, nta);
    return dt == TW_F16 ? pick_mode_t<TW_F16, false, EW>(mode, ms, ncb, nta) : pick_mode_t<TW_BF16, false, EW>(mode, ms, ncb, nta);
}
template <bool EW>
const void* pick_kernel_of(int dt, int mode, int ms, int ncb, bool fused, bool nta) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_mode<TW_F16, true, EW>(mode, ms, ncb, nta) : pick_mode<TW_BF16, true, EW>(mode, ms, ncb, nta);
    return dt == TW_F16 ? pick_mode<TW_F16, false, EW>(mode, ms, ncb, nta) : pick_mode<TW_BF16, false, EW>(mode, ms, ncb, nta);
}
// (ew: the blob carries an element-wise residual)
const void* pick_kernel_t(int dt, int mode, int ms, int ncb, bool fused, bool nta, bool ew) {
    return ew ? pick_kernel_t_of<true>(dt, mode, ms, ncb, fused, nta) : pick_kernel_t_of<false>(dt, mode, ms, ncb, fused, nta);
}
const void* pick_kernel(int dt, int mode, int ms, int ncb, bool fused, bool nta, bool ew) {
    return ew ? pick_kernel_of<true>(dt, mode, ms, ncb, fused, nta) : pick_kernel_of<false>(dt, mode, ms, ncb, fused, nta);
}
const void* pick_team_kernel(int dt, int ncb, bool fused, bool transposed) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_team<TW_F16, true>(ncb, transposed) : pick_team<TW_BF16, true>(ncb, transposed);
    return dt == TW_F16 ? pick_team<TW_F16, false>(ncb, transposed) : pick_team<TW_BF16, false>(ncb, transposed);
}
const void* pick_narrow_kernel(int dt, int ncb, bool fused) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_narrow<TW_F16, true>(ncb) : pick_narrow<TW_BF16, true>(ncb);
    return dt == TW_F16 ? pick_narrow<TW_F16, false>(ncb) : pick_narrow<TW_BF16, false>(ncb);
}
const void* pick_stream_kernel(int dt, int ncb, bool fused) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_stream<TW_F16, true>(ncb) : pick_stream<TW_BF16, true>(ncb);
    return dt == TW_F16 ? pick_stream<TW_F16, false>(ncb) : pick_stream<TW_BF16, false>(ncb);
}
const void* pick_rows_kernel(int dt, int ncb, bool fused, int stages) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_rows<TW_F16, true>(ncb, stages) : pick_rows<TW_BF16, true>(ncb, stages);
    return dt == TW_F16 ? pick_rows<TW_F16, false>(ncb, stages) : pick_rows<TW_BF16, false>(ncb, stages);
}
const void* pick_reduce_kernel(int dt, int ncb, bool fused, bool transposed) {
    using namespace tw_parts;
    if (fused) return dt == TW_F16 ? pick_reduce<TW_F16, true>(ncb, transposed) : pick_reduce<TW_BF16, true>(ncb, transposed);
    return dt == TW_F16 ? pick_reduce<TW_F16, false>(ncb, transposed) : pick_reduce<TW_BF16, false>(ncb, transposed);
}

// Per-device facts looked up once (the entries are written with the same value by every thread
// that races to fill them, so no lock is needed).
constexpr int kMaxDevices = 64;
std::atomic<int> g_cus[kMaxDevices];

int current_device() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
    return dev;
}

int device_cus(int dev) {
    int n = g_cus[dev].load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return -1;
    g_cus[dev].store(n, std::memory_order_relaxed);
    return n;
}

// The dynamic-LDS limit of a kernel is raised to the hardware maximum once per (device, kernel).
constexpr int kMaxKernels = 560;
std::atomic<unsigned> g_lds_set[kMaxDevices][kMaxKernels];

int ensure_lds(int dev, int kernel_id, const void* fn) {
    if (g_lds_set[dev][kernel_id].load(std::memory_order_acquire)) return TW_OK;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsLimit) != hipSuccess)
        return TW_ERR_HIP;
    g_lds_set[dev][kernel_id].store(1u, std::memory_order_release);
    return TW_OK;
}

// the numbers of the kernels that pick_kernel, pick_kernel_t and pick_team_kernel give
int tile_kernel_id(const TwHeader* h, const Plan& pl, int kmode, bool fused, bool nta, bool transposed) {
    const int variant = pl.team_shift > 0 ? 8 : kmode == 0 ? (pl.ms == 2 ? 0 : 1) : 2 * kmode + (nta ? 0 : 1);   // 0..8
    return (h->ew_nnz > 0 ? 240 : 0) + (transposed ? 120 : 0) + (fused ? 60 : 0) + (h->dtype == TW_F16 ? 0 : 30) + 3 * variant +
           (h->ncb == 4 ? 0 : h->ncb == 2 ? 1 : 2);
}

}  // namespace

extern "C" int tw_gemm_workspace(const void* blob_host, int M, size_t* ws_bytes) {
    if (!blob_host || !ws_bytes || M < 0) return TW_ERR_ARG;
    const TwHeader* h = (const TwHeader*)blob_host;
    if (h->magic != TW_MAGIC || h->version != TW_FORMAT_VERSION) return TW_ERR_BUF;
    // the counters, and behind them the partial results of a split-K plan (the larger of the two boundaries'), as
    // planned for the current GPU (256 compute units when there is none to ask)
    size_t need = 256;
    if (M > 0 && h->T > 0 && h->n_chunks > 1) {
        int n_cu = 256;
        const int dev = current_device();
        if (dev >= 0 && device_cus(dev) > 0) n_cu = device_cus(dev);
        for (int tr = 0; tr < 2; ++tr) {
            Plan pl;
            if (make_plan(h, M, n_cu, pl, tr != 0) == TW_OK && 256 + pl.partial_bytes > need) need = 256 + pl.partial_bytes;
        }
    }
    *ws_bytes = need;
    return TW_OK;
}

extern "C" int tw_gemm_plan(const void* blob_host, int M, int n_cu, int transposed, tw_plan_t* plan) {
    if (!blob_host || !plan || M < 0 || n_cu <= 0) return TW_ERR_ARG;
    const TwHeader* h = (const TwHeader*)blob_host;
    if (h->magic != TW_MAGIC || h->version != TW_FORMAT_VERSION) return TW_ERR_BUF;
    memset(plan, 0, sizeof(*plan));
    if (M == 0 || h->T == 0) return TW_OK;      // nothing to multiply: a fill kernel at most
    Plan pl;
    const int rc = make_plan(h, M, n_cu, pl, transposed != 0);
    if (rc) return rc;
    plan->mode = pl.mode;
    plan->rows_per_block = pl.row_step;
    plan->tiles_per_set = pl.tiles_per_set;
    plan->n_row_blocks = pl.n_mblocks;
    plan->n_sets = pl.n_seg;
    plan->n_items = pl.n_items;
    plan->grid = pl.n_items < n_cu ? pl.n_items : n_cu;
    plan->lds_bytes = !transposed && parts_by_direct_loads(h, h->K, pl) ? part_lds_bytes() : pl.lds_bytes;
    plan->row_lists = pl.urow_off != 0;
    plan->k_parts = pl.n_parts;
    plan->team_waves = 1 << pl.team_shift;
    if (transposed) {
        plan_rows(h, M, ((long)M + 7) / 8 * 8, n_cu, pl, false);
        if (pl.rows_group > 0) {
            plan->tile_items = (int32_t)(((long)M + (h->ncb == 4 ? 127 : 255)) / (h->ncb == 4 ? 128 : 256) * h->T);
            plan->tile_lds_bytes = pl.rows_lds;
        }
    }
    return TW_OK;
}

extern "C" int tw_gemm(const void* blob_host, const void* blob_dev, const void* A, int M, int lda, void* C,
                       int ldc, void* workspace, size_t ws_bytes, void* hip_stream) {
    return tw_gemm_bias_act(blob_host, blob_dev, A, M, lda, nullptr, TW_ACT_NONE, C, ldc, workspace, ws_bytes,
                            hip_stream);
}

namespace {
// what tw_gemm and its variants on the row-major boundary refuse before anything is enqueued
int check_gemm_args(const void* blob_host, const void* blob_dev, const void* A, int M, int lda, const void* bias,
                    tw_act act, const void* C, int ldc, const void* workspace, size_t ws_bytes) {
    if (!blob_host || !blob_dev || !A || !C || !workspace || M < 0) return TW_ERR_ARG;
    if (act != TW_ACT_NONE && act != TW_ACT_RELU && act != TW_ACT_GELU) return TW_ERR_ARG;
    if (((uintptr_t)bias & 1) != 0) return TW_ERR_ALIGN;
    const TwHeader* h = (const TwHeader*)blob_host;
    if (h->magic != TW_MAGIC || h->version != TW_FORMAT_VERSION) return TW_ERR_BUF;
    if (ws_bytes < 256) return TW_ERR_BUF;
    if (lda < h->K || ldc < h->N) return TW_ERR_ARG;
    if ((lda & 7) != 0 || ((uintptr_t)A & 15) != 0 || ((uintptr_t)C & 1) != 0) return TW_ERR_ALIGN;
    if (((uintptr_t)blob_dev & 255) != 0 || ((uintptr_t)workspace & 255) != 0) return TW_ERR_ALIGN;
    return TW_OK;
}

// ---- scratch memory of the entry point that allocates nothing and takes no workspace (tw_gemm_static) ----
// The scheduler's counters (its first 256 bytes) and the fp32 partial results of a split-K plan (the rest; the
// planner takes a split only if they fit) live in this array instead of a buffer of the caller.  Only the counters
// need a defined start value; the partial results are written before they are read.  Every GPU holds its own
// copy at its own address; host code must use the address that hipGetSymbolAddress returns with that GPU
// current (the array's name is only a host-side stand-in), so it is looked up once per device and kept.
__device__ __align__(256) unsigned char tw_static_scratch[TW_STATIC_SCRATCH_BYTES];
std::atomic<void*> g_static_scratch[kMaxDevices];

int static_scratch(int dev, void** out) {
    void* ptr = g_static_scratch[dev].load(std::memory_order_acquire);
    if (!ptr) {
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(tw_static_scratch)) != hipSuccess || !ptr) return TW_ERR_HIP;
        g_static_scratch[dev].store(ptr, std::memory_order_release);
    }
    *out = ptr;
    return TW_OK;
}

// the counters start every call at zero, whatever an earlier call left behind (a kernel, not a memset: the
// call may be recorded into a graph)
__global__ void tw_clear_kernel(unsigned* w, int n) {
    if ((int)threadIdx.x < n) w[threadIdx.x] = 0u;
}
}  // namespace

extern "C" int tw_gemm_static(const void* blob_host, const void* blob_dev, const void* A, int M, int lda, void* C,
                              int ldc, void* hip_stream) {
    const int dev = current_device();
    if (dev < 0) return TW_ERR_HIP;
    void* scratch = nullptr;
    int rc = static_scratch(dev, &scratch);
    if (rc) return rc;
    rc = check_gemm_args(blob_host, blob_dev, A, M, lda, nullptr, TW_ACT_NONE, C, ldc, scratch, TW_STATIC_SCRATCH_BYTES);
    if (rc) return rc;
    if (M == 0) return TW_OK;
    unsigned* w_ = (unsigned*)scratch;
    int n_ = 64;
    void* cargs[] = {(void*)&w_, (void*)&n_};
    if (hipLaunchKernel((const void*)tw_clear_kernel, dim3(1), dim3(64), cargs, 0, (hipStream_t)hip_stream) != hipSuccess)
        return TW_ERR_HIP;
    return tw_gemm_bias_act(blob_host, blob_dev, A, M, lda, nullptr, TW_ACT_NONE, C, ldc, scratch, TW_STATIC_SCRATCH_BYTES,
                            hip_stream);
}

extern "C" int tw_gemm_bias_act(const void* blob_host, const void* blob_dev, const void* A, int M, int lda,
                                const void* bias, tw_act act, void* C, int ldc, void* workspace, size_t ws_bytes,
                                void* hip_stream) {
    {
        const int rc0 = check_gemm_args(blob_host, blob_dev, A, M, lda, bias, act, C, ldc, workspace, ws_bytes);
        if (rc0) return rc0;
    }
    const TwHeader* h = (const TwHeader*)blob_host;
    if (M == 0) return TW_OK;
    hipStream_t stream = (hipStream_t)hip_stream;

    if (h->T == 0) {
        const long total = (long)M * h->N;
        int blocks = (int)((total + 255) / 256);
        if (blocks > 4096) blocks = 4096;
        unsigned short* c_ = (unsigned short*)C;
        long ldc_ = ldc;
        int m_ = M, n_ = h->N, act_ = (int)act;
        const unsigned short* bias_ = (const unsigned short*)bias;
        void* fargs[] = {(void*)&c_, (void*)&ldc_, (void*)&m_, (void*)&n_, (void*)&bias_, (void*)&act_};
        const void* ffn = h->dtype == TW_F16 ? (const void*)tw_fill_kernel<TW_F16> : (const void*)tw_fill_kernel<TW_BF16>;
        if (hipLaunchKernel(ffn, dim3(blocks), dim3(256), fargs, 0, stream) != hipSuccess) return TW_ERR_HIP;
        return launch_xcols(h, blob_dev, A, lda, C, ldc, M, bias, (int)act, false, stream);
    }

    const int dev = current_device();
    if (dev < 0) return TW_ERR_HIP;
    const int n_cu = device_cus(dev);
    if (n_cu <= 0) return TW_ERR_HIP;
    Plan pl;
    int rc = make_plan(h, M, n_cu, pl, false, ws_bytes, act == TW_ACT_GELU);
    if (rc) return rc;
    plan_stream(h, lda, pl);
    const bool split = pl.n_parts > 1;
    const bool fused_epilogue = bias != nullptr || act != TW_ACT_NONE;
    const bool fused = fused_epilogue && !split;      // split K: the epilogue is the second kernel's
    // streamed K: the activations carry the streaming hint only when one workgroup reads a row block's rows
    const bool nta = pl.mode == 0 || pl.n_seg == 1;
    const int kmode = split ? 3 : pl.mode;             // the kernel's MODE
    const bool bf16 = h->dtype != TW_F16;
    // the kernel that runs, its number among those whose on-chip memory limit is raised once, and its on-chip memory
    const void* fn;
    int kernel_id;
    unsigned lds_bytes = pl.lds_bytes;
    if (pl.stream_items > 0) {
        fn = pick_stream_kernel(h->dtype, h->ncb, fused);
        kernel_id = 492 + (bf16 ? 6 : 0) + (fused ? 3 : 0) + (h->ncb >> 1);
        lds_bytes = stream_lds_bytes();
    } else if (parts_by_direct_loads(h, lda, pl)) {
        fn = bf16 ? tw_parts::pick_part<TW_BF16>(h->ncb, pl.tiles_per_set) : tw_parts::pick_part<TW_F16>(h->ncb, pl.tiles_per_set);
        kernel_id = 528 + (bf16 ? 9 : 0) + (pl.tiles_per_set <= 2 ? 0 : pl.tiles_per_set <= 4 ? 3 : 6) + (h->ncb >> 1);
        lds_bytes = part_lds_bytes();
    } else if (pl.narrow) {
        fn = pick_narrow_kernel(h->dtype, h->ncb, fused);
        kernel_id = 516 + (bf16 ? 6 : 0) + (fused ? 3 : 0) + (h->ncb >> 1);
    } else {
        const bool team = pl.team_shift > 0;
        fn = team ? pick_team_kernel(h->dtype, h->ncb, fused, false) : pick_kernel(h->dtype, kmode, pl.ms, h->ncb, fused, nta, h->ew_nnz > 0);
        kernel_id = tile_kernel_id(h, pl, kmode, fused, nta, false);
    }
    if (!fn) return TW_ERR_UNSUPPORTED;
    const void* fn_reduce = nullptr;
    if (split) {
        fn_reduce = pick_reduce_kernel(h->dtype, h->ncb, fused_epilogue, false);
        if (!fn_reduce) return TW_ERR_UNSUPPORTED;
    }
    rc = ensure_lds(dev, kernel_id, fn);
    if (rc) return rc;

    TwGemmParams p;
    p.blob = (const unsigned char*)blob_dev;
    p.A = (const unsigned short*)A;
    p.C = (unsigned short*)C;
    p.counters = (int*)workspace;
    p.bias = (const unsigned short*)bias; p.act = (int)act;
    p.lda = lda; p.ldc = ldc;
    p.M = M; p.K = h->K; p.N = h->N; p.T = h->T;
    p.k_chunk = h->k_chunk; p.n_chunks = h->n_chunks; p.G = h->G;
    p.n_mblocks = pl.n_mblocks; p.n_seg = pl.n_seg; p.n_items = pl.n_items; p.tiles_per_set = pl.tiles_per_set; p.row_step = pl.row_step;
    p.at_pitch = pl.at_pitch; p.abuf_bytes = pl.abuf_bytes;
    p.stage_off = pl.stage_off; p.misc_off = pl.misc_off;
    p.off_sched_desc = h->off_sched_desc; p.off_step_ptr = h->off_step_ptr; p.off_goff = h->off_goff;
    p.off_dpos = h->off_dpos; p.off_bvals = h->off_bvals;
    p.off_zero_ptr = h->off_zero_ptr; p.off_zero_cols = h->off_zero_cols;
    p.off_urow = h->off_urow; p.off_ucnt = h->off_ucnt;
    p.urow_off = pl.stream_items > 0 ? p.stage_off + kStreamTiles * kStageBytes : 0;   // tw_stream_kernel's ring
    p.off_ew_ptr = h->off_ew_ptr; p.off_ew_goff = h->off_ew_goff; p.off_ew_b = h->off_ew_b; p.has_ew = h->ew_nnz > 0;
    p.off_xm_ptr = h->off_xm_ptr; p.off_xm_goff = h->off_xm_goff; p.off_xm_b = h->off_xm_b; p.off_zero_xc = h->off_zero_xc;
    p.stream_stores = ((uintptr_t)C & 127) == 0 && (ldc & 63) == 0;
    p.off_xc_tile_ptr = h->off_xc_tile_ptr; p.off_xc_col = h->off_xc_col; p.off_xc_ptr = h->off_xc_ptr;
    p.off_xc_k = h->off_xc_k; p.off_xc_v = h->off_xc_v; p.xbuf_off = pl.xbuf_off;
    p.n_parts = pl.n_parts; p.chunks_per_part = pl.chunks_per_part; p.team_shift = pl.team_shift;
    p.partials = (float*)((unsigned char*)workspace + 256);
    const int grid = pl.n_items < n_cu ? pl.n_items : n_cu;
    void* args[] = {(void*)&p};
    if (hipLaunchKernel(fn, dim3(grid), dim3(kThreads), args, lds_bytes, stream) != hipSuccess) return TW_ERR_HIP;
    if (split) {
        const long units = (long)pl.n_mblocks * h->T * 8;                 // a wave per pass of a tile
        if (hipLaunchKernel(fn_reduce, dim3((unsigned)units), dim3(64), args, 0, stream) != hipSuccess) return TW_ERR_HIP;
    }
    return launch_xcols(h, blob_dev, A, lda, C, ldc, M, bias, (int)act, false, stream, pl.xbuf_off != 0);
}

extern "C" int tw_gemm_t(const void* blob_host, const void* blob_dev, const void* At, int M, int ldat, void* Ct,
                         int ldct, void* workspace, size_t ws_bytes, void* hip_stream) {
    return tw_gemm_t_bias_act(blob_host, blob_dev, At, M, ldat, nullptr, TW_ACT_NONE, Ct, ldct, workspace, ws_bytes,
                              hip_stream);
}

extern "C" int tw_gemm_t_bias_act(const void* blob_host, const void* blob_dev, const void* At, int M, int ldat,
                                  const void* bias, tw_act act, void* Ct, int ldct, void* workspace, size_t ws_bytes,
                                  void* hip_stream) {
    if (!blob_host || !blob_dev || !At || !Ct || !workspace || M < 0) return TW_ERR_ARG;
    if (act != TW_ACT_NONE && act != TW_ACT_RELU && act != TW_ACT_GELU) return TW_ERR_ARG;
    if (((uintptr_t)bias & 1) != 0) return TW_ERR_ALIGN;
    const bool fused_epilogue = bias != nullptr || act != TW_ACT_NONE;
    const TwHeader* h = (const TwHeader*)blob_host;
    if (h->magic != TW_MAGIC || h->version != TW_FORMAT_VERSION) return TW_ERR_BUF;
    if (ws_bytes < 256) return TW_ERR_BUF;
    if (ldat < M || ldct < M) return TW_ERR_ARG;
    if ((ldat & 7) != 0 || (ldct & 7) != 0 || ((uintptr_t)At & 15) != 0 || ((uintptr_t)Ct & 15) != 0) return TW_ERR_ALIGN;
    if (((uintptr_t)blob_dev & 255) != 0 || ((uintptr_t)workspace & 255) != 0) return TW_ERR_ALIGN;
    if (M == 0) return TW_OK;
    hipStream_t stream = (hipStream_t)hip_stream;

    if (h->T == 0) {   // every row of Ct is zero
        const long total = (long)h->N * M;
        int blocks = (int)((total + 255) / 256);
        if (blocks > 4096) blocks = 4096;
        unsigned short* c_ = (unsigned short*)Ct;
        long ldc_ = ldct;
        int n_ = h->N, m_ = M, act_ = (int)act;
        const unsigned short* bias_ = (const unsigned short*)bias;
        void* fargs[] = {(void*)&c_, (void*)&ldc_, (void*)&n_, (void*)&m_, (void*)&bias_, (void*)&act_};
        const void* ffn = h->dtype == TW_F16 ? (const void*)tw_fill_rows_kernel<TW_F16> : (const void*)tw_fill_rows_kernel<TW_BF16>;
        if (hipLaunchKernel(ffn, dim3(blocks), dim3(256), fargs, 0, stream) != hipSuccess) return TW_ERR_HIP;
        return launch_xcols(h, blob_dev, At, ldat, Ct, ldct, M, bias, (int)act, true, stream);
    }

    const int dev = current_device();
    if (dev < 0) return TW_ERR_HIP;
    const int n_cu = device_cus(dev);
    if (n_cu <= 0) return TW_ERR_HIP;
    Plan pl;
    int rc = make_plan(h, M, n_cu, pl, /*transposed=*/true, ws_bytes, act == TW_ACT_GELU);
    if (rc) return rc;
    plan_rows(h, M, ldat, n_cu, pl, act == TW_ACT_GELU);
    const bool split = pl.n_parts > 1;
    const bool fused = fused_epilogue && !split;      // split K: the epilogue is the second kernel's
    const bool nta = pl.mode == 0 || pl.n_seg == 1;
    const int kmode = split ? 3 : pl.mode;             // the kernel's MODE
    // the kernel that runs and its number among those whose on-chip memory limit is raised once
    const void* fn;
    int kernel_id;
    if (pl.rows_group > 0) {
        fn = pick_rows_kernel(h->dtype, h->ncb, fused, pl.rows_stages);
        kernel_id = pl.rows_stages == 8 ? 480 + (fused ? 6 : 0) + (h->dtype == TW_F16 ? 0 : 3) + (h->ncb >> 1) : -1;   // (at most 64 KB with four)
    } else {
        const bool team = pl.team_shift > 0;
        fn = team ? pick_team_kernel(h->dtype, h->ncb, fused, true) : pick_kernel_t(h->dtype, kmode, pl.ms, h->ncb, fused, nta, h->ew_nnz > 0);
        kernel_id = tile_kernel_id(h, pl, kmode, fused, nta, true);
    }
    if (!fn) return TW_ERR_UNSUPPORTED;
    const void* fn_reduce = nullptr;
    if (split) {
        fn_reduce = pick_reduce_kernel(h->dtype, h->ncb, fused_epilogue, true);
        if (!fn_reduce) return TW_ERR_UNSUPPORTED;
    }
    if (kernel_id >= 0) rc = ensure_lds(dev, kernel_id, fn);
    if (rc) return rc;

    TwGemmParams p;
    p.blob = (const unsigned char*)blob_dev;
    p.A = (const unsigned short*)At;
    p.C = (unsigned short*)Ct;
    p.counters = (int*)workspace;
    p.bias = (const unsigned short*)bias; p.act = (int)act;
    p.lda = ldat; p.ldc = ldct;
    p.M = M; p.K = h->K; p.N = h->N; p.T = h->T;
    p.k_chunk = h->k_chunk; p.n_chunks = h->n_chunks; p.G = h->G;
    p.n_mblocks = pl.n_mblocks; p.n_seg = pl.n_seg; p.n_items = pl.n_items; p.tiles_per_set = pl.tiles_per_set; p.row_step = pl.row_step;
    p.at_pitch = pl.at_pitch; p.abuf_bytes = pl.abuf_bytes;
    p.stage_off = pl.stage_off; p.misc_off = pl.misc_off;
    p.off_sched_desc = h->off_sched_desc; p.off_step_ptr = h->off_step_ptr; p.off_goff = h->off_goff;
    p.off_dpos = h->off_dpos; p.off_bvals = h->off_bvals;
    p.off_zero_ptr = h->off_zero_ptr; p.off_zero_cols = h->off_zero_cols;
    p.off_urow = h->off_urow; p.off_ucnt = h->off_ucnt;
    p.off_ew_ptr = h->off_ew_ptr; p.off_ew_goff = h->off_ew_goff; p.off_ew_b = h->off_ew_b; p.has_ew = h->ew_nnz > 0;
    p.off_xm_ptr = h->off_xm_ptr; p.off_xm_goff = h->off_xm_goff; p.off_xm_b = h->off_xm_b; p.off_zero_xc = h->off_zero_xc;
    p.urow_off = pl.urow_off;
    p.off_xc_tile_ptr = h->off_xc_tile_ptr; p.off_xc_col = h->off_xc_col; p.off_xc_ptr = h->off_xc_ptr;
    p.off_xc_k = h->off_xc_k; p.off_xc_v = h->off_xc_v; p.xbuf_off = pl.xbuf_off;
    p.stream_stores = ((uintptr_t)Ct & 127) == 0 && (ldct & 63) == 0;
    p.n_parts = pl.n_parts; p.chunks_per_part = pl.chunks_per_part; p.team_shift = pl.team_shift;
    p.partials = (float*)((unsigned char*)workspace + 256);
    const unsigned lds_bytes = pl.lds_bytes;
    const int grid = pl.n_items < n_cu ? pl.n_items : n_cu;
    void* args[] = {(void*)&p};
    if (pl.rows_group > 0) {
        const int bt = h->ncb == 4 ? rows_bt<4>() : rows_bt<1>();
        p.n_mblocks = (M + bt - 1) / bt; p.rows_group = pl.rows_group;
        return hipLaunchKernel(fn, dim3((unsigned)(p.n_mblocks * h->T)), dim3(256), args, pl.rows_lds, stream) == hipSuccess ? TW_OK : TW_ERR_HIP;
    }
    if (hipLaunchKernel(fn, dim3(grid), dim3(kThreads), args, lds_bytes, stream) != hipSuccess) return TW_ERR_HIP;
    if (split) {
        const long units = (long)pl.n_mblocks * h->T * h->ncb;            // a wave per column block of a tile
        if (hipLaunchKernel(fn_reduce, dim3((unsigned)units), dim3(64), args, 0, stream) != hipSuccess) return TW_ERR_HIP;
    }
    return launch_xcols(h, blob_dev, At, ldat, Ct, ldct, M, bias, (int)act, true, stream, pl.xbuf_off != 0);
}

// ---- the transposes at the two ends of a network that runs on the transposed boundary (Sec. VI) ----
namespace {
__global__ __launch_bounds__(256) void tw_transpose_kernel(const unsigned short* src, long lds_, int rows, int cols,
                                                           unsigned short* dst, long ldd, int vec) {
    // 64 x 64 tile through LDS, kept TRANSPOSED there: tile[c][r], rows of 144 bytes (16-byte aligned pieces, and
    // consecutive rows 4 banks apart)
    constexpr int kPitch = 144;
    __shared__ __attribute__((aligned(16))) unsigned char tile[64 * kPitch];
    const int c0 = blockIdx.x * 64, r0 = blockIdx.y * 64;
    const int t = threadIdx.x;
    if (vec && r0 + 64 <= rows && c0 + 64 <= cols) {
        // whole tile, 16-byte aligned rows on both sides: 16-byte loads and stores, 2-byte LDS writes in between
        const int j = t & 7;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = (t >> 3) + 32 * i;
            const tw_u32x4 v = tw_load16_stream(src + (long)(r0 + r) * lds_ + c0 + 8 * j);   // read once, written once
            const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                *(unsigned short*)(tile + (8 * j + e) * kPitch + r * 2) = (unsigned short)(w[e >> 1] >> (16 * (e & 1)));
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int c = (t >> 3) + 32 * i;
            // (rows of dst on 128-byte boundaries: the eight lanes of a row write a whole line)
            if (vec == 2) tw_store16_stream(dst + (long)(c0 + c) * ldd + r0 + 8 * j, *(const tw_u32x4*)(tile + c * kPitch + j * 16));
            else *(tw_u32x4*)tw_opaque(dst + (long)(c0 + c) * ldd + r0 + 8 * j) = *(const tw_u32x4*)(tile + c * kPitch + j * 16);
        }
        return;
    }
    // edge tiles and unaligned matrices: element by element
    const int tx = t & 63, ty = t >> 6;
    for (int r = ty; r < 64; r += 4)
        if (r0 + r < rows && c0 + tx < cols) *(unsigned short*)(tile + tx * kPitch + r * 2) = src[(long)(r0 + r) * lds_ + c0 + tx];
    __syncthreads();
    for (int c = ty; c < 64; c += 4)
        if (c0 + c < cols && r0 + tx < rows) dst[(long)(c0 + c) * ldd + r0 + tx] = *(const unsigned short*)(tile + c * kPitch + tx * 2);
}
}  // namespace

extern "C" int tw_transpose(const void* src, int ld_src, int rows, int cols, void* dst, int ld_dst, void* hip_stream) {
    if (!src || !dst || rows < 0 || cols < 0 || ld_src < cols || ld_dst < rows) return TW_ERR_ARG;
    if (((uintptr_t)src & 1) != 0 || ((uintptr_t)dst & 1) != 0) return TW_ERR_ALIGN;
    if (rows == 0 || cols == 0) return TW_OK;
    const long gx = ((long)cols + 63) / 64, gy = ((long)rows + 63) / 64;
    if (gy > 65535) return TW_ERR_UNSUPPORTED;
    int vec = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0 && (ld_src & 7) == 0 && (ld_dst & 7) == 0;
    if (vec && ((uintptr_t)dst & 127) == 0 && (ld_dst & 63) == 0) vec = 2;
    const unsigned short* s_ = (const unsigned short*)src;
    unsigned short* d_ = (unsigned short*)dst;
    long lds2 = ld_src, ldd2 = ld_dst;
    int vec_ = vec;
    void* targs[] = {(void*)&s_, (void*)&lds2, (void*)&rows, (void*)&cols, (void*)&d_, (void*)&ldd2, (void*)&vec_};
    return hipLaunchKernel((const void*)tw_transpose_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(256), targs, 0,
                           (hipStream_t)hip_stream) == hipSuccess ? TW_OK : TW_ERR_HIP;
}
#endif  // host code
