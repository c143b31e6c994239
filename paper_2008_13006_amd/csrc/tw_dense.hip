// tw_dense_gemm: C = A . B, the dense yardstick of the TW kernel (the paper's baseline is a tiled
// dense GEMM on the matrix unit, Sec. IV-A Fig. 4 step 1 and Sec. VI "Tiling").  Same MFMA
// instruction, same operand roles, same epilogue as tw_gemm; B is ordinary row-major K x N.
//
// Workgroup: a (64 * MSW) x 256 block of C, 8 waves as 2 (rows) x 4 (columns), wave tile (32 * MSW) x 64;
// MSW = 4 (256 rows), 2 or 1, chosen per call (the paper's tiling leaves the thread-block shape to the
// implementation, Sec. VI "Tiling").  Workgroups are persistent and walk blocks of C.
//
// K advances 64 at a time through a ring of LDS buffers that loads fill DIRECTLY (buffer_load .. lds): a staged K step
// costs no registers and no LDS write instructions, so a whole step of loads is in flight while another is
// multiplied, and the ring runs on into the workgroup's next block of C: its first step lands during this one's
// last steps and its epilogue.  Direct loads write 1 KB of consecutive LDS per wave instruction, so rows cannot be padded;
// bank conflicts are avoided by WHICH 16-byte piece of a row a lane fetches instead (kept at slot piece ^ f(row)).
// What bounds it: the matrix units under the card's power limit.  16384 x 768 x 3072 in fp16: 81 us (950 TFLOP/s; 95 us with
// the operands staged through registers).  Parts left out, measured at 83 us for the whole: without loads and stores 55, with
// the MFMAs alone 50 (1560 TFLOP/s), and 72 us as it is on operands of zeros, where the clock stays up; the loads cost 14
// us and the stores 15.  On 16384 x 3072 x 768 80 us (95 through registers), 8192 x 4096 x 1024 74 (88), 2048 x 3072 x 768 31
// (57), 1500 x 1000 x 2000 14.5 (31).
// Spreading a step's requests over its MFMAs instead of one burst behind the barrier: no gain on real operands.
//
// The operands of contraction slots 16*ks+16 .. are read from LDS before the MFMAs of slots 16*ks .. are issued,
// across the K step's barrier too (it sits in front of the last 8 MFMAs of a step).
#include <hip/hip_runtime.h>

#include <atomic>

#include "../../include/tw.h"
#include "tw_device.hpp"
#include "tw_pieces.h"

namespace {

typedef short tw_i16x4 __attribute__((ext_vector_type(4)));
constexpr int kThreads = 512;
constexpr int BN = 256, KB = 64, KS = KB / 16;
constexpr int B_BYTES = KB * BN * 2;   // 32768
// MSW: 32-row blocks of a wave's tile; the workgroup's block has BM = 64 * MSW rows
template <int MSW> constexpr int bm_of() { return 64 * MSW; }
template <int MSW> constexpr int a_bytes_of() { return bm_of<MSW>() * KB * 2; }             // 32768 for 256 rows
template <int MSW> constexpr int buf_bytes_of() { return a_bytes_of<MSW>() + B_BYTES; }
// Buffers of the ring: as many as fit (128, 144, 120 KB of LDS).  (Steps of 32 K positions in four or five buffers, with
// three or four steps on their way, measured the same as two buffers of 64: what bounds the loop is not the latency.)
template <int MSW> constexpr int stages_of() { return MSW == 4 ? 2 : 3; }
// Behind the ring: the last, ragged 16-byte piece of A's last row and of B's (they are read element by element, once)
constexpr int kEndBytes = 32;
template <int MSW> constexpr int lds_bytes_of() { return stages_of<MSW>() * buf_bytes_of<MSW>() + kEndBytes; }
constexpr int kDenseStage = 4096;   // bytes of a wave's staging area in the epilogue: the areas lie in the buffer of the last step
static_assert(8 * kDenseStage <= buf_bytes_of<1>(), "the epilogue's staging areas fit one buffer of the ring");

struct DenseParams {
    const unsigned short* A;
    const unsigned short* B;
    unsigned short* C;
    long lda, ldb, ldc;
    int M, N, K;
    int nbm, nbn;
    const unsigned short* bias;   // N values added before the activation, or null
    int act;                      // tw_act
    int stream;                   // rows of C start on 128-byte boundaries: whole lines go out as streaming stores
};

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
// The same value, as one the compiler cannot compute with ahead of time: addresses of the epilogue are then formed there
// and not kept in registers (or in scratch memory) through the whole loop.
__device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Offsets at and above this are out of a buffer descriptor's range: such a lane fetches zeros.
constexpr unsigned kRange = 0x80000000u;
__device__ const unsigned tw_dense_zeros[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ void load_lds_wide(const void* src, unsigned lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void lds_meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ tw_u32x4 descriptor(const unsigned short* base) {
    const uint64_t a = (uint64_t)base;
    return tw_u32x4{(unsigned)uni((int)(unsigned)a), (unsigned)uni((int)(unsigned)(a >> 32)) & 0xFFFFu, kRange, 0x00020000u};
}

// the t-th block of C: four row blocks are walked together, so that the workgroups of one XCD (neighbouring t) share
// rows of A and columns of B in its L2.  (One, two, four, eight together: the same on full batches, 512 x 768 x 3072 11.0, 10.35,
// 10.3, 10.3 us, 300 x 130 x 66000 25.1, 26.1, 24.4, 24.6, 16384 x 3072 x 768 82.3, 83.4, 82.5, 83.5.)
__device__ __forceinline__ void block_of(const DenseParams& p, int t, int bm, int& m0, int& n0) {
    const int per = 4 * p.nbn, g = t / per, rem = t - g * per;
    const int gm = p.nbm - 4 * g < 4 ? p.nbm - 4 * g : 4;
    const int nb = rem / gm;
    m0 = (4 * g + rem - nb * gm) * bm;
    n0 = nb * BN;
}

// Hands the bias of the wave's 64 columns (`own`: this lane's column) round through its staging area: lane half h receives
// the columns 32*cb + 8*q + 4*h + 0..3 as bias[cb][q].  Once per block of C, before the area takes results.
__device__ __forceinline__ void spread_bias(unsigned short own, unsigned char* stage, int lane, tw_u32x2 (&bias)[2][4]) {
    asm volatile("" ::: "memory");
    *(unsigned short*)(stage + 2 * lane) = own;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[cb][q] = *(const tw_u32x2*)(stage + 64 * cb + 16 * q + 8 * (lane >> 5));
    asm volatile("" ::: "memory");
}

// Adds the bias and applies the activation, in place, to a 32 x 64 block: lane l holds row l%32 and of acc[cb] the
// columns 32*cb + 8*(r/4) + 4*(l/32) + r%4.  The activation is chosen once per block, so that each choice is straight-line
// code.  (A branch and a load of the bias for every element: 32 round trips to memory per block, each behind the
// stores and the next block's requests: 16384 x 768 x 3072 took 121 us with a bias and 126 with GELU, this way 84 and
// 100, 512 x 768 x 3072 14.7 and 15.3, this way 10.7 and 12.4; without a fused epilogue they take 84 and 10.3.)
template <int DT>
__device__ __forceinline__ void add_bias_act(tw_f32x16 (&acc)[2], const tw_u32x2 (&bias)[2][4], int act) {
    auto value = [&](int cb, int r) {
        const unsigned two = bias[cb][r >> 2][(r >> 1) & 1];
        return acc[cb][r] + tw_to_f32<DT>((unsigned short)(r & 1 ? two >> 16 : two));
    };
    if (act == TW_ACT_GELU) {                                // uniform
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][r] = tw_gelu(value(cb, r));
    } else if (act == TW_ACT_RELU) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float x = value(cb, r);
                acc[cb][r] = x > 0.f ? x : 0.f;
            }
    } else {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][r] = value(cb, r);
    }
}

// Writes one 32 x 64 block of a wave's results to C[row0 .., col0 .. col0 + width) through the wave's staging area of
// 32 rows x 128 bytes.  Column octet c of row r lies at slot c ^ (r/2 % 8) of the row, its two halves swapped in
// rows 16..31: the 8-byte writes of 32 lanes (32 rows, one octet) and the 16-byte reads (8 rows, 8 octets) then both
// use every bank once.  stream: whole 128-byte lines may be written with streaming stores.
// The LDS executes a wave's instructions in order: fences for the compiler are enough.
template <int DT>
__device__ __forceinline__ void store_block(const tw_f32x16 (&acc)[2], unsigned char* stage, unsigned short* C, long ldc,
                                            int row0, int M, int col0, int width, int lane, bool stream) {
    const int mrow = lane & 31, h = lane >> 5;
    asm volatile("" ::: "memory");
    unsigned char* myrow = stage + mrow * 128 + (h ^ (mrow >> 4)) * 8;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            tw_u32x2 v;
            v.x = (unsigned)tw_cvt<DT>(acc[cb][4 * q]) | ((unsigned)tw_cvt<DT>(acc[cb][4 * q + 1]) << 16);
            v.y = (unsigned)tw_cvt<DT>(acc[cb][4 * q + 2]) | ((unsigned)tw_cvt<DT>(acc[cb][4 * q + 3]) << 16);
            *(tw_u32x2*)(myrow + (((4 * cb + q) ^ ((mrow >> 1) & 7)) << 4)) = v;
        }
    asm volatile("" ::: "memory");
    // 8 lanes cover the 64 columns of a row, 8 rows per pass
    const int j = lane & 7;
    tw_u32x4 v[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int r = (lane >> 3) + 8 * p;
        v[p] = *(const tw_u32x4*)(stage + r * 128 + ((j ^ ((r >> 1) & 7)) << 4));
        if (p >= 2) v[p] = tw_u32x4{v[p].z, v[p].w, v[p].x, v[p].y};
    }
    asm volatile("" ::: "memory");
    unsigned short* dst = C + (long)(row0 + (lane >> 3)) * ldc + col0 + 8 * j;
    const int rows = M - row0 - (lane >> 3);
    if (width == 64 && stream) {                               // wave-uniform
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (8 * p < rows) tw_store16_stream(dst + (long)(8 * p) * ldc, v[p]);
    } else {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if (8 * p >= rows) continue;
            unsigned short* d = tw_opaque(dst) + (long)(8 * p) * ldc;
            if (8 * j + 8 <= width) *(tw_u32x4_a2*)d = v[p];
            else if (8 * j < width) {                          // the row's ragged end
                const unsigned e[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
                for (int i = 0; i < 7; ++i)
                    if (8 * j + i < width) d[i] = (unsigned short)(e[i >> 1] >> (16 * (i & 1)));
            }
        }
    }
}

// NTA: the activations are read by one column of blocks only (N <= 256), so they carry the streaming hint.
// WIDE: row pitches for which a block's offsets do not fit a buffer descriptor (64-bit addresses per lane instead).
template <int DT, int MSW, bool NTA, bool WIDE>
__global__ __launch_bounds__(kThreads) void tw_dense_kernel(const DenseParams p) {
    constexpr int BM = bm_of<MSW>(), A_BYTES = a_bytes_of<MSW>(), BUF_BYTES = buf_bytes_of<MSW>(), NST = stages_of<MSW>();
    constexpr int kLoads = MSW + 4;               // requests of a wave per K step
    // 16-byte piece u of row r of A lies at slot u ^ fa(r) of the row: any 16 lanes that a 16-byte LDS read serves
    // together then hit 16 different slots of the banks
    auto fa = [](int r) { return (r >> 1) & 7; };
    extern __shared__ __attribute__((aligned(128))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int h = lane >> 5, l32 = lane & 31;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // workgroups that land on the same XCD (ids equal modulo 8) get neighbouring blocks of C
    const int total = p.nbm * p.nbn, grid = (int)gridDim.x;
    int bid = blockIdx.x;
    if ((grid & 7) == 0) bid = (bid & 7) * (grid >> 3) + (bid >> 3);
    const int nk = (p.K - 1) / KB + 1;

    // What this lane fetches of a step.  A: request i brings rows 8*(wave + 8*i) + lane/8.  B: request i brings K rows
    // 2*(wave + 8*i) + lane/32, slot lane%32 of a row holds piece slot ^ 4*(row % 4) ^ 2*(row/8 % 2): the rows of a
    // transposing read then lie in different parts of the banks, whichever 32 lanes are served together.
    const int ra = 8 * wave + (lane >> 3);
    const int ua = (lane & 7) ^ fa(ra);
    const int rb = 2 * wave + h;
    auto fb = [](int r) { return ((r & 3) << 2) ^ (((r >> 3) & 1) << 1); };
    const int ub = l32 ^ fb(rb);

    // the request cursor: step ck of block ct, running ahead of the multiplication
    int ct = bid, ck = 0, cm0, cn0;
    block_of(p, ct, BM, cm0, cn0);
    // rows up to which this lane's piece is there to be read: of A in the last K step (in the others its pieces are whole), of
    // B in the block's columns; counted from the lane's first row
    const int a_last = tw_piece_rows((nk - 1) * KB + ua * 8, p.M, p.K) - ra;
    int b_rows = tw_piece_rows(cn0 + ub * 8, p.K, p.N) - rb;
    auto issue = [&](int buf) {
        const unsigned dst = lds0 + (unsigned)uni(buf) * BUF_BYTES;
        const int k0 = ck * KB;
        const int am = (ck == nk - 1 ? a_last : p.M - ra) - cm0, bm = b_rows - k0;
        if constexpr (WIDE) {
#pragma unroll
            for (int i = 0; i < MSW; ++i) {
                const int r = ra + 64 * i;
                const void* src = 64 * i < am ? (const void*)(p.A + (long)(cm0 + r) * p.lda + (k0 + ua * 8)) : (const void*)tw_dense_zeros;
                load_lds_wide(src, dst + (unsigned)(wave + 8 * i) * 1024u);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = rb + 16 * i;
                const void* src = 16 * i < bm ? (const void*)(p.B + (long)(k0 + r) * p.ldb + (cn0 + ub * 8)) : (const void*)tw_dense_zeros;
                load_lds_wide(src, dst + A_BYTES + (unsigned)(wave + 8 * i) * 1024u);
            }
        } else {
            const tw_u32x4 da = descriptor(p.A + (long)cm0 * p.lda + k0);
            const tw_u32x4 db = descriptor(p.B + (long)k0 * p.ldb + cn0);
            const unsigned lda2 = 2u * (unsigned)p.lda, ldb2 = 2u * (unsigned)p.ldb;
#pragma unroll
            for (int i = 0; i < MSW; ++i) {
                const int r = ra + 64 * i;
                tw_load_lds<NTA>(da, 64 * i < am ? (unsigned)r * lda2 + ua * 16 : kRange, dst + (unsigned)(wave + 8 * i) * 1024u);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = rb + 16 * i;
                tw_load_lds<false>(db, 16 * i < bm ? (unsigned)r * ldb2 + ub * 16 : kRange, dst + A_BYTES + (unsigned)(wave + 8 * i) * 1024u);
            }
        }
        if (++ck == nk) {
            ck = 0;
            ct += grid;
            if (ct < total) {
                block_of(p, ct, BM, cm0, cn0);
                b_rows = tw_piece_rows(cn0 + ub * 8, p.K, p.N) - rb;
            } else {                                         // nothing more to read
                cm0 = p.M;
                b_rows = 0;
            }
        }
    };

    // where this lane's operands lie in a buffer
    const int j = lane & 15;
    const unsigned oa = (unsigned)(wm * 32 * MSW + l32) * 128u + (unsigned)((h ^ fa(l32)) << 4);
    // weight operand by transposing reads of the K-major B tile: in each 16-lane block, lane j addresses K row
    // 8h + 4r + j/4 at the four columns 4*(j%4) .. of the block's 16 columns
    const unsigned ob = A_BYTES + (unsigned)(8 * h + (j >> 2)) * 512u +
                        (unsigned)(((wn * 8 + ((lane >> 4) & 1) * 2 + ((j & 3) >> 1)) ^ ((j >> 2) << 2) ^ (h << 1)) * 16 + (j & 1) * 8);
    tw_u16x8 w[2][2], a[2][MSW];
    auto fetch = [&](int slot, const unsigned char* buf, int ks) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const unsigned char* lb = buf + (ob ^ (unsigned)(cb * 64)) + ks * 16 * 512;
            const tw_i16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) tw_i16x4*)(lb));
            const tw_i16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) tw_i16x4*)(lb + 4 * 512));
            w[slot][cb] = tw_u16x8{(unsigned short)lo4[0], (unsigned short)lo4[1], (unsigned short)lo4[2], (unsigned short)lo4[3],
                                   (unsigned short)hi4[0], (unsigned short)hi4[1], (unsigned short)hi4[2], (unsigned short)hi4[3]};
        }
#pragma unroll
        for (int ms = 0; ms < MSW; ++ms) a[slot][ms] = *(const tw_u16x8*)(buf + (oa ^ (unsigned)(ks << 5)) + ms * 4096);
    };
    // The last K step of the block at (m0, n0), where K or N is no multiple of 8.  What the last 16-byte piece of A's rows
    // holds beyond K belongs to the row's pitch and counts as zero; the last row's ragged piece is not read by the ring.
    unsigned char* const ends = smem + NST * BUF_BYTES;
    const int kr = p.K & 7, nr = p.N & 7;
    auto mend_ends = [&](unsigned char* buf, int kt, int m0, int n0) {
        if (kt == nk - 1 && (kr != 0 || (nr != 0 && p.N - n0 < BN))) {      // uniform
            if (kr != 0 && tid < BM) {
                unsigned char* piece = buf + tid * 128 + ((((p.K & 63) >> 3) ^ fa(tid)) << 4);
                if (m0 + tid == p.M - 1) *(tw_u32x4*)piece = *(const tw_u32x4*)ends;
                else for (int e = kr; e < 8; ++e) *(unsigned short*)(piece + 2 * e) = 0;
            }
            if (nr != 0 && p.N - n0 < BN && tid == kThreads - 1) {
                const int r = (p.K - 1) & 63;
                *(tw_u32x4*)(buf + A_BYTES + r * (BN * 2) + ((((p.N - n0) >> 3) ^ fb(r)) << 4)) = *(const tw_u32x4*)(ends + 16);
            }
            lds_meet();
        }
    };

    tw_f32x16 acc[MSW][2];
    auto multiply = [&](int slot) {
#pragma unroll
        for (int ms = 0; ms < MSW; ++ms)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb) acc[ms][cb] = tw_mfma<DT>(w[slot][cb], a[slot][ms], acc[ms][cb]);
    };

#pragma unroll
    for (int i = 0; i < NST; ++i) issue(i);
    if ((kr | nr) != 0 && tid < 16) {                        // lanes 0..7: A's end, 8..15: B's
        const int e = tid & 7;
        unsigned short v = 0;
        if (tid < 8 && e < kr) v = p.A[(long)(p.M - 1) * p.lda + (p.K - kr + e)];
        if (tid >= 8 && e < nr) v = p.B[(long)(p.K - 1) * p.ldb + (p.N - nr + e)];
        *(unsigned short*)(ends + 2 * tid) = v;
    }
    int pos = 0;                                             // buffer of the current step
    int m0, n0;                                              // block of C
    block_of(p, bid, BM, m0, n0);
    tw_lds_wait<(NST - 1) * kLoads>();
    mend_ends(smem, 0, m0, n0);
    fetch(0, smem, 0);
    for (int t = bid; t < total; t += grid) {
#pragma unroll
        for (int ms = 0; ms < MSW; ++ms)
#pragma unroll
            for (int cb = 0; cb < 2; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[ms][cb][r] = 0.f;
        for (int kt = 0;; ++kt) {
            unsigned char* cur = smem + pos * BUF_BYTES;
            const int npos = pos + 1 == NST ? 0 : pos + 1;
            unsigned char* nxt = smem + npos * BUF_BYTES;
#pragma unroll
            for (int ks = 0; ks < KS - 1; ++ks) {
                fetch((ks + 1) & 1, cur, ks + 1);
                __builtin_amdgcn_sched_barrier(0);
                multiply(ks & 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (kt + 1 == nk) break;
            // the next step has landed and every wave has read this one: its buffer takes the step after the ring's last
            // (the operands are read before the requests' address arithmetic, not behind it: 36.1 -> 31.6 us on 2048 x 3072 x 768)
            tw_lds_wait<(NST - 2) * kLoads>();
            mend_ends(nxt, kt + 1, m0, n0);
            fetch(0, nxt, 0);
            __builtin_amdgcn_sched_barrier(0);
            issue(pos);
            __builtin_amdgcn_sched_barrier(0);
            multiply(1);
            __builtin_amdgcn_sched_barrier(0);
            pos = npos;
        }
        const int col0 = n0 + wn * 64;
        const int width = (p.N - col0) < 64 ? (p.N - col0) : 64;
        const bool fused = p.bias != nullptr || p.act != TW_ACT_NONE;
        unsigned short own_bias = 0;                         // of the column col0 + lane, asked for ahead of the last MFMAs
        const int elane = fresh(lane);
        if (p.bias != nullptr && elane < width) own_bias = p.bias[col0 + elane];
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        tw_lds_wait<(NST - 2) * kLoads>();
        // epilogue through per-wave staging areas in the buffer of the last step; the next block's first steps are landing in the others
        {
            unsigned char* stage = smem + pos * BUF_BYTES + wave * kDenseStage;
            if (width > 0) {
                tw_u32x2 bias[2][4];
                if (fused) spread_bias(own_bias, stage, elane, bias);
#pragma unroll
                for (int ms = 0; ms < MSW; ++ms) {
                    if (fused) add_bias_act<DT>(acc[ms], bias, p.act);
                    store_block<DT>(acc[ms], stage, p.C, p.ldc, m0 + wm * 32 * MSW + ms * 32, p.M, col0, width, elane, p.stream != 0);
                }
            }
        }
        if (t + grid >= total) break;
        lds_meet();
        issue(pos);
        pos = pos + 1 == NST ? 0 : pos + 1;
        block_of(p, t + grid, BM, m0, n0);
        mend_ends(smem + pos * BUF_BYTES, 0, m0, n0);
        fetch(0, smem + pos * BUF_BYTES, 0);
    }
    // requests of the ring may still be on their way to this workgroup's LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int MSW>
const void* pick(tw_dtype dt, bool nta, bool wide) {
    if (wide) return dt == TW_F16 ? (const void*)tw_dense_kernel<TW_F16, MSW, false, true> : (const void*)tw_dense_kernel<TW_BF16, MSW, false, true>;
    if (dt == TW_F16) return nta ? (const void*)tw_dense_kernel<TW_F16, MSW, true, false> : (const void*)tw_dense_kernel<TW_F16, MSW, false, false>;
    return nta ? (const void*)tw_dense_kernel<TW_BF16, MSW, true, false> : (const void*)tw_dense_kernel<TW_BF16, MSW, false, false>;
}

}  // namespace

extern "C" int tw_dense_gemm(const void* A, int lda, const void* B, int ldb, void* C, int ldc, int M, int N, int K,
                             tw_dtype dt, void* hip_stream) {
    return tw_dense_gemm_bias_act(A, lda, B, ldb, nullptr, TW_ACT_NONE, C, ldc, M, N, K, dt, hip_stream);
}

extern "C" int tw_dense_gemm_bias_act(const void* A, int lda, const void* B, int ldb, const void* bias, tw_act act,
                                      void* C, int ldc, int M, int N, int K, tw_dtype dt, void* hip_stream) {
    if (!A || !B || !C || M < 0 || N <= 0 || K <= 0) return TW_ERR_ARG;
    if (act != TW_ACT_NONE && act != TW_ACT_RELU && act != TW_ACT_GELU) return TW_ERR_ARG;
    if (((uintptr_t)bias & 1) != 0) return TW_ERR_ALIGN;
    if (dt != TW_F16 && dt != TW_BF16) return TW_ERR_ARG;
    if (lda < K || ldb < N || ldc < N) return TW_ERR_ARG;
    if ((lda & 7) || (ldb & 7) || (ldc & 7)) return TW_ERR_ALIGN;
    if (((uintptr_t)A & 15) || ((uintptr_t)B & 15) || ((uintptr_t)C & 15)) return TW_ERR_ALIGN;
    if (M == 0) return TW_OK;
    DenseParams p;
    p.A = (const unsigned short*)A; p.B = (const unsigned short*)B; p.C = (unsigned short*)C;
    p.lda = lda; p.ldb = ldb; p.ldc = ldc;
    p.M = M; p.N = N; p.K = K;
    p.bias = (const unsigned short*)bias; p.act = (int)act;
    p.stream = ((uintptr_t)C & 127) == 0 && (ldc & 63) == 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TW_ERR_HIP;
    static std::atomic<int> n_cus[64];
    int n_cu = n_cus[dev].load(std::memory_order_relaxed);
    if (n_cu <= 0) {
        if (hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu <= 0) return TW_ERR_HIP;
        n_cus[dev].store(n_cu, std::memory_order_relaxed);
    }
    // Rows per block: 256, 128 or 64, whichever needs the least time by a simple model: rounds of workgroups
    // times the block height, with 25 % (80 %) on top for the lower blocks, which read the weights more often.
    // (768 -> 768 at M = 16384 makes 192 blocks of 256 rows: one round at three quarters of the chip beats the
    // two rounds of 128-row blocks; 4096 -> 1024 at M = 8192 makes 128 blocks: 128-row blocks fill the chip.)
    p.nbn = (N - 1) / BN + 1;
    int msw = 4;
    double best = 0.0;
    for (int cand = 4; cand >= 1; cand >>= 1) {
        const long blk = (long)((M + 64L * cand - 1) / (64 * cand)) * p.nbn;
        const double cost = (double)((blk + n_cu - 1) / n_cu) * cand * (cand == 4 ? 1.0 : cand == 2 ? 1.25 : 1.8);
        if (cand == 4 || cost < best) { best = cost; msw = cand; }
    }
    p.nbm = (int)((M + 64L * msw - 1) / (64 * msw));
    const long blocks = (long)p.nbm * p.nbn;
    if (blocks > 0x7fffffffL) return TW_ERR_UNSUPPORTED;
    const void* fn;
    int lds;
    // offsets of a block (256 rows of A, 64 of B) must fit 31 bits for the kernels that address through a descriptor
    const bool wide = 256L * lda >= (1L << 30) || 64L * ldb >= (1L << 30);
    const bool nta = p.nbn == 1 && !wide;
    if (msw == 4) { fn = pick<4>(dt, nta, wide); lds = lds_bytes_of<4>(); }
    else if (msw == 2) { fn = pick<2>(dt, nta, wide); lds = lds_bytes_of<2>(); }
    else { fn = pick<1>(dt, nta, wide); lds = lds_bytes_of<1>(); }
    static std::atomic<unsigned char> lds_set[64][2][15];
    const int slot = 3 * msw + (wide ? 2 : nta ? 1 : 0);
    if (!lds_set[dev][dt][slot].load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return TW_ERR_HIP;
        lds_set[dev][dt][slot].store(1, std::memory_order_release);
    }
    void* args[] = {(void*)&p};
    return hipLaunchKernel(fn, dim3((unsigned)(blocks < n_cu ? blocks : n_cu)), dim3(kThreads), args, lds, (hipStream_t)hip_stream) == hipSuccess
               ? TW_OK : TW_ERR_HIP;
}
