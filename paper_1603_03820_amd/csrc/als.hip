// One ALS half-sweep on gfx950 (MI355X): C ABI of include/als.h plus its kernels.
//
// Per row u of a CSR matrix (eq. 2 of the paper; Algorithm 1's Get_Hermitian_X then
// Batch_Solve):  A_u = sum theta_v theta_v^T + lambda n_u I,  b_u = sum r_uv theta_v,
// x_u = A_u^{-1} b_u.
//
// Design (one wave = one worker):
//   k_plan          integer partition of the rows (and of long rows' entries) into chunks of a
//                   cost axis: W large chunks, then 8W small ones (see als_plan in als.h); no
//                   host synchronisation needed.
//   k_herm_solve    persistent waves take chunks in order and walk their row pieces; gather theta_v
//                   for 32 entries at a time straight into MFMA operand layout (lane = 16*k +
//                   column, so each group of 16 lanes reads 64 contiguous bytes of one theta_v),
//                   with the rating appended as column f, split every value into three bf16 parts
//                   that add up to it exactly, and accumulate the upper block-triangle of the
//                   augmented Gram matrix [A b; b^T c] in fp32 with six
//                   v_mfma_f32_16x16x32_bf16 per tile (three for the mostly-padding last block
//                   column, an FMA per value when it holds the rating alone).  Rows that end in
//                   the chunk are regularised and solved in registers by a blocked Cholesky: per
//                   16-column block, the 16 x 16 diagonal tile is factored and inverted with lane
//                   broadcasts, and the panel and trailing updates are 16x16x4 fp32 MFMAs; the
//                   forward substitution rides along as the augmented column; the back
//                   substitution is a short blocked pass.
//   k_reduce_*      rows cut by chunk boundaries: sum the chunks' partial accumulators in chunk
//                   order (fixed, so results are reproducible), then the same solve.
//   k_rmse_rows     residuals per stored entry through the same gather pipeline, x_u held in
//                   registers per row piece; fp64 partial sums in a fixed order.
//
// Register layout of the accumulators (the 16x16 MFMA C/D layout): tile (I,J), I <= J, lane l,
// element r holds M[16 I + 4 (l >> 4) + r][16 J + (l & 15)] of the augmented matrix M, whose
// column f is b (and M[f][f] = sum r^2, unused).  NB = f/16 + 1 column blocks cover f + 1.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <climits>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "als.h"

typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int kWave = 64;
constexpr int kMaxNB = ALS_F_MAX / 16 + 1;      // 9 column blocks of 16 cover f + 1 <= 129
constexpr int kSnap = 256;                      // partition cut grid (entries)
constexpr int kCostPerEntry = 16;               // c_nnz
constexpr int kTailDiv = 8;                     // the small chunks cover floor(T / 8) of the cost
constexpr int kSmallPerWave = 8;                // small chunks per wave
constexpr int chunks_of(int waves) { return waves * (1 + kSmallPerWave); }
constexpr int kMaxWavesPerCU = 32;
constexpr int kRmseWavesPerCU = 32;                // RMSE: up to 8 waves per SIMD (occupancy)
constexpr int kTransposeWavesPerCU = 8;            // CSR -> CSC: row blocks per CU (at most)

constexpr int ntiles(int nb) { return nb * (nb + 1) / 2; }
// upper block-triangle, row-major: tile (I, J) with I <= J
constexpr int tu(int nb, int I, int J) { return I * nb - I * (I - 1) / 2 + (J - I); }
// floats per partial-accumulator slot: tiles, 4 per lane
constexpr int slot_floats(int nb) { return ntiles(nb) * 4 * kWave; }

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

// acc + a' * b, where a' is `a` taken from lane N of the lane's 16-lane row (DPP row_newbcast:N),
// in one v_fmac.  The only vector instruction here that is inline assembly, around which the compiler
// inserts no wait states.  A DPP source needs two of them after its last VALU write; the caller keeps
// them (volatile, so the statements stay in source order and the caller can count).  A matrix
// instruction's result needs ten; factor_tile keeps those.  (As update_dpp and an FMA it becomes a DPP
// move for two FMAs and up to 20 registers more: ranks up to 16 lose a resident wave or two, f = 16
// 326 -> 365 us on 20M ratings of 200,000 users, f = 32 on the movie user side 1.79 -> 1.86 ms; f = 128
// and short rows gain 1%.)  `a` may be the value of `acc` itself: as an operand of its own, a copy
// the register allocator makes for the tied accumulator never becomes the DPP source.
template <int N>
__device__ __forceinline__ float fmac_bcast(float acc, float a, float b) {
    asm volatile("v_fmac_f32_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc)
                 : "v"(a), "v"(b), "n"(N));
    return acc;
}
// Two wait states (for a DPP read of a register a VALU op wrote just before).
__device__ __forceinline__ void dpp_settle() { asm volatile("s_nop 1"); }

// v taken from the lane that DPP control CTRL names (every lane of the row has one).
template <int CTRL>
__device__ __forceinline__ float dpp_take(float v) {
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// Whether this lane's bit is set in a constant 64-bit lane mask.
__device__ __forceinline__ bool in_lanes(uint64_t mask) {
    return __builtin_amdgcn_inverse_ballot_w64(mask);
}

// Sum over the 16 lanes of a DPP row (lanes 16g..16g+15), returned to all 16 lanes with the
// same bits: swap neighbours, swap pairs (quad_perm), then mirror within 8 and within 16.
__device__ __forceinline__ float row_sum16(float v) {
    v += dpp_f<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_f<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_f<0x141>(v);   // row_half_mirror
    v += dpp_f<0x140>(v);   // row_mirror
    return v;
}

// Sums over the 16 lanes of a DPP row of v[0..3], transposed: lane c of the row returns the sum
// of v[c & 3] (each sum lands in four lanes, added in different orders).  Pairs of values trade
// halves between neighbours (xor 1), then between pairs (xor 2), so every lane keeps adding one
// value; rotations by 4 and 8 finish the sum.  11 VALU ops against 16 for four plain row sums.
__device__ __forceinline__ float row_sum16_t(f4 v) {
    const bool odd = in_lanes(0xAAAAAAAAAAAAAAAAull), two = in_lanes(0xCCCCCCCCCCCCCCCCull);
    const float a0 = (odd ? v[1] : v[0]) + dpp_take<0xB1>(odd ? v[0] : v[1]);   // quad_perm [1,0,3,2]
    const float a2 = (odd ? v[3] : v[2]) + dpp_take<0xB1>(odd ? v[2] : v[3]);
    float s = (two ? a2 : a0) + dpp_take<0x4E>(two ? a0 : a2);                  // quad_perm [2,3,0,1]
    s += dpp_take<0x124>(s);                                                    // row_ror:4
    s += dpp_take<0x128>(s);                                                    // row_ror:8
    return s;
}

// ------------------------------------------------------------------------------- plan ----

// How the persistent waves of k_herm_solve come by their chunks.  Atomics on one address are
// performed one after the other, about 11.5 ns each on this part: with one counter the 9W
// successful and W failing claims of a half-sweep took 0.47 ms at W = 4,096 (f = 16 and 40: all of
// the time of a call on 50,000 or 1M ratings), and the waves' first claims alone 25-47 us.  So
//   - a short sweep (at most static_entries entry equivalents of cost per wave) claims nothing: wave
//     w runs large chunk w and the eight small chunks W + 8w .. W + 8w + 7, an equal share of the
//     cost;
//   - a longer one, whose waves finish at different times, claims from kStripes counters on lines
//     of their own: stripe s holds chunks s, s + kStripes, ... in order, for the waves of blocks
//     b with b / 8 = s (mod kStripes), which lie on all XCDs (block b runs on XCD b mod 8).  A
//     stripe's 64 or more waves (W = 1,024 at f = 128) even it out among themselves, so none goes on to
//     another stripe
//     (looking at the other counters at the end made the kernel twice as long).
constexpr int kStripes = 16;                    // a power of two
constexpr int kStripeWords = 64;                // 256 bytes apart
// Fixed shares against claims, 10M, 6M and 4M cost entries at f = 16, 40 and 100 (2,048 a wave): 134
// against 157, 212 against 223, 561 against 522 us; a quarter of that: 58, 88, 211 against 91, 110,
// 212; four times: 445, 722, 1,921 against 438, 686, 1,774.
constexpr int64_t kStaticEntries = 2048;        // up to 3 column blocks
constexpr int64_t static_entries(int nb) { return nb <= 3 ? kStaticEntries : kStaticEntries / 4; }

// Cost prefix P(u) = c_nnz rowptr[u] + c_row u, T = P(m).  C chunks: W large ones cover
// T1 = T - T2 and C - W small ones the tail T2 = floor(T / kTailDiv) (T2 = 0 when C = W);
// boundary b sits at s_b = floor(T1 b / W) for b <= W, T1 + floor(T2 (b - W) / (C - W)) beyond.
// The first threads also reset the counters the persistent waves claim chunks from and the flag of
// rows set aside (see kTinyX).
__global__ void k_plan(const int64_t* __restrict__ rowptr, int64_t m, int W, int C, int64_t c_nnz,
                       int64_t c_row, int64_t q, int64_t* __restrict__ bounds,
                       unsigned* __restrict__ chunk_ctr, unsigned* __restrict__ set_aside) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < kStripes && chunk_ctr) chunk_ctr[b * kStripeWords] = 0u;
    if (b == 0 && set_aside) *set_aside = 0u;
    if (b > C) return;
    const int64_t T = c_nnz * rowptr[m] + c_row * m;
    const int64_t T2 = C > W ? T / kTailDiv : 0, T1 = T - T2;
    int64_t s;   // floor(X b / D) as Q b + floor(R b / D), without 128-bit products
    if (b <= W) {
        s = T1 / W * b + (T1 % W) * b / W;
    } else {
        const int64_t D = C - W, e = b - W;
        s = T1 + T2 / D * e + (T2 % D) * e / D;
    }
    int64_t lo = 0, hi = m;                  // largest u in [0, m] with P(u) <= s
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (c_nnz * rowptr[mid] + c_row * mid <= s) lo = mid; else hi = mid - 1;
    }
    const int64_t u = lo;
    int64_t kk = 0;
    if (u < m) {
        const int64_t nu = rowptr[u + 1] - rowptr[u];
        const int64_t over = s - (c_nnz * rowptr[u] + c_row * u) - c_row;
        int64_t raw = over <= 0 ? 0 : (over + c_nnz - 1) / c_nnz;
        if (raw > nu) raw = nu;
        kk = (raw + q / 2) / q * q;
        if (kk > 0 && kk + q / 2 > nu) kk = nu;
    }
    bounds[2 * b] = u;
    bounds[2 * b + 1] = kk;
}

// --------------------------------------------------------------------- Gram + RHS --------

// Gather pipeline of the RMSE: the gathers of step s + kDepth are issued before step s runs, so every gather
// has kDepth steps of matrix work of this wave to hide behind.  Steps run in unrolled groups of
// kGroup = kDepth + 1 with as many operand buffers; at sub-step J the step kDepth ahead goes into
// the buffer whose step ran at sub-step J - 1, so the buffers rotate by renaming, never by copying
// registers that are loading.  Each entry's gather word and rating come in batches of 48 entries
// (12 steps) through a two-slot LDS ring (entry p of the piece sits at p mod 96): batch k+1 is
// loaded (one entry per lane) at the top of batch k's first group and stored at the top of its
// second group, before the first gather that reads it (which needs kDepth <= 5) and after the
// last one that read the slot's previous batch, so any register carried around the loop only
// ever waits on a load older than the gathers in flight.
constexpr int kDepth = 3;
constexpr int kGroup = kDepth + 1;
constexpr int kBatch = 48;
constexpr int kBatchGroups = kBatch / 4 / kGroup;
constexpr int kRing = 2 * kBatch;
static_assert(kBatchGroups * kGroup * 4 == kBatch && kBatchGroups >= 2 && 2 * kDepth <= 11,
              "pipeline depth must divide the batch and stay within one group of lookahead");

// The last block column NB-1 holds q = f - 16 (NB-1) + 1 real columns, the last theta columns and
// the rating; the rest of it is padding.  Its form (LAST):
//   kLastRating  q = 1, the rating alone (f a multiple of 16): no operand block; the rating column is
//                one fp32 FMA per gathered value;
//   kLastPacked  q <= 5: lane c holds column c mod q, the real columns three times over, for the
//                three parts of the split below;
//   kLastTiles   otherwise: lane c holds column c, an ordinary block.
constexpr int kLastTiles = 0, kLastPacked = 1, kLastRating = 2, kLastForms = 3;
constexpr int kPackedColumns = 5;
constexpr int last_form(int f) {
    return f % 16 == 0 ? kLastRating : (f % 16 + 1 <= kPackedColumns ? kLastPacked : kLastTiles);
}
__device__ __forceinline__ int packed_column(int c, int q) { return c < 3 * q ? c % q : 16; }

// The theta gather of one step, as MFMA operands: lane (g, c) of block I reads
// theta_{v_g}[16 I + c] (of a packed last block: the column of packed_column), and the lanes of
// column f take the rating.  Three forms (the second template argument):
//   kFormBuffer, for theta below 2 GiB: raw buffer loads against a descriptor that bounds
//     theta.  The gather word of an entry is its byte offset 4 f v; an entry past the piece's end
//     gets the buffer size, and the lanes of padding columns add the size to their offset, so
//     those loads return 0 by the hardware's range check and nothing is masked in the loop.
//   kFormGlobal, for any size: 64-bit global loads; the gather word is the row's address (a row
//     of zeros past the piece's end), and padding lanes read a column of their block's cache
//     line whose value is then replaced (see Gather<NB, kFormGlobal, P>).
//   kFormStaged, a design alternative kept for the ablation: the rows go through LDS.
// All issue their loads unconditionally, so they stay in flight across earlier matrix ops.
constexpr int kFormGlobal = 0, kFormBuffer = 1, kFormStaged = 2;

// One entry of the index ring: the entry's gather word (a byte offset or a row address, as the
// gather form defines it) and its rating.
template <class W>
struct RingEntryT {
    W e;
    float r;
};

template <int NB, int BUF, int LAST = kLastTiles>
struct Gather;

template <int NB, int LAST>
struct Gather<NB, kFormBuffer, LAST> {
    using Entry = RingEntryT<int>;
    static constexpr int kBlocks = LAST == kLastRating ? NB - 1 : NB;   // operand values per step
    static constexpr int kBuf = kBlocks;                                // gathered values per step
    __amdgpu_buffer_rsrc_t rs;
    unsigned fbytes, size, lo, llast;
    bool jr;
    __device__ __forceinline__ Gather(const float* theta, int64_t n, int f, int c,
                                      float* = nullptr) {
        fbytes = 4u * (unsigned)f;
        size = (unsigned)n * fbytes;
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(theta), 0, (int)size,
                                               0x00020000);
        lo = 4u * (unsigned)c;
        const int jlast = 16 * (NB - 1) + (LAST == kLastPacked ? packed_column(c, f - 16 * (NB - 1) + 1) : c);
        llast = jlast < f ? 4u * (unsigned)jlast : size;
        jr = jlast == f;
    }
    __device__ __forceinline__ int word(int col, bool valid) const {
        return valid ? (int)((unsigned)col * fbytes) : (int)size;
    }
    __device__ __forceinline__ void issue(int e, float (&v)[kBuf]) const {
        const unsigned base = (unsigned)e + lo;
#pragma unroll
        for (int I = 0; I < NB - 1; ++I)
            v[I] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rs, base + 64u * I, 0, 0));
        if constexpr (LAST != kLastRating)
            v[NB - 1] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(rs, (unsigned)e + llast, 0, 0));
    }
    __device__ __forceinline__ void operands(const float (&B)[kBuf], float r,
                                             float (&v)[kBlocks]) const {
#pragma unroll
        for (int I = 0; I < NB - 1; ++I) v[I] = B[I];
        if constexpr (LAST != kLastRating) v[NB - 1] = jr ? r : B[NB - 1];
    }
};

// A row of zeros, read in place of theta_v by the 64-bit gather for entries past a piece's end.
__device__ float g_zero_row[16 * kMaxNB];

// Gather<NB, kFormGlobal, LAST>, for any size of theta: 64-bit global loads.  The gather word of an
// entry is its row's address (g_zero_row past the piece's end, so such entries gather zeros);
// lane (g, c) reads block I < NB-1 at that address + 4 (16 I + c), with 64 I as the
// instruction's immediate offset.  In the last block a padding lane reads a column of the cache
// line the block's real lanes read -- its first column, or column f - 1 when it has none -- and
// the value is replaced (by the rating in column f, else by 0).
template <int NB, int LAST>
struct Gather<NB, kFormGlobal, LAST> {
    using Entry = RingEntryT<uint64_t>;
    static constexpr int kBlocks = LAST == kLastRating ? NB - 1 : NB;
    static constexpr int kBuf = kBlocks;
    typedef const __attribute__((address_space(1))) float* gptr;
    uint64_t base, zero;
    unsigned fbytes, lo, llast;
    bool jpad, jr;
    __device__ __forceinline__ Gather(const float* theta, int64_t, int f, int c,
                                      float* = nullptr) {
        base = (uint64_t)theta;
        zero = (uint64_t)g_zero_row;
        fbytes = 4u * (unsigned)f;
        lo = 4u * (unsigned)c;
        const int jlast = 16 * (NB - 1) + (LAST == kLastPacked ? packed_column(c, f - 16 * (NB - 1) + 1) : c);
        jpad = jlast >= f;
        const int jsame = 16 * (NB - 1) < f ? 16 * (NB - 1) : f - 1;
        llast = 4u * (unsigned)(jpad ? jsame : jlast);
        jr = jlast == f;
    }
    __device__ __forceinline__ uint64_t word(int col, bool valid) const {
        return valid ? base + (uint64_t)(unsigned)col * fbytes : zero;
    }
    __device__ __forceinline__ void issue(uint64_t e, float (&v)[kBuf]) const {
        const gptr pl = (gptr)(e + lo);
#pragma unroll
        for (int I = 0; I < NB - 1; ++I) v[I] = pl[16 * I];
        if constexpr (LAST != kLastRating) v[NB - 1] = *(gptr)(e + llast);
    }
    __device__ __forceinline__ void operands(const float (&B)[kBuf], float r,
                                             float (&v)[kBlocks]) const {
#pragma unroll
        for (int I = 0; I < NB - 1; ++I) v[I] = B[I];
        if constexpr (LAST != kLastRating) v[NB - 1] = jpad ? (jr ? r : 0.f) : B[NB - 1];
    }
};

// Gather<NB, kFormStaged>: a design alternative (for the ablation of the gather; theta below
// 2 GiB, f a multiple of 4): the step's four theta rows are read row by row with two 16-byte
// loads per lane -- lane (g, c) reads bytes 16 c and 256 + 16 c of row g, the rating lane's
// bytes included -- written to a per-wave LDS buffer of four rows of 16 NB floats (zero past
// the loaded columns), and the MFMA operands are read back from it (lane (g, c) of block I:
// row g, column 16 I + c).  Past the piece's end and past a row's 4 f bytes the loads are out of
// range and return zeros, as in the buffer form.
constexpr int stage_floats(int nb) { return 4 * 16 * nb; }

template <int NB>
struct Gather<NB, kFormStaged, kLastTiles> {
    using Entry = RingEntryT<int>;
    static constexpr int kBlocks = NB, kBuf = 8;
    __amdgpu_buffer_rsrc_t rs;
    unsigned fbytes, size, o0, o1;
    int lane;
    bool jr;
    float* stage;
    __device__ __forceinline__ Gather(const float* theta, int64_t n, int f, int c, float* st) {
        fbytes = 4u * (unsigned)f;
        size = (unsigned)n * fbytes;
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(theta), 0, (int)size,
                                               0x00020000);
        o0 = 16u * c < fbytes ? 16u * c : size;
        o1 = 256u + 16u * c < fbytes ? 256u + 16u * c : size;
        jr = 16 * (NB - 1) + c == f;
        lane = (int)(threadIdx.x & 63);
        stage = st;
    }
    __device__ __forceinline__ int word(int col, bool valid) const {
        return valid ? (int)((unsigned)col * fbytes) : (int)size;
    }
    __device__ __forceinline__ void issue(int e, float (&v)[kBuf]) const {
        const f4 a = __builtin_bit_cast(
            f4, __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)e + o0, 0, 0));
        const f4 b = __builtin_bit_cast(
            f4, __builtin_amdgcn_raw_buffer_load_b128(rs, (unsigned)e + o1, 0, 0));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = a[j];
            v[4 + j] = b[j];
        }
    }
    __device__ __forceinline__ void operands(const float (&B)[kBuf], float r,
                                             float (&v)[NB]) const {
        const int g = lane >> 4, c = lane & 15;
        float* row = stage + g * 16 * NB;
        if (4 * c + 4 <= 16 * NB)
            *reinterpret_cast<f4*>(row + 4 * c) = f4{B[0], B[1], B[2], B[3]};
        if (64 + 4 * c + 4 <= 16 * NB)
            *reinterpret_cast<f4*>(row + 64 + 4 * c) = f4{B[4], B[5], B[6], B[7]};
        __syncthreads();
#pragma unroll
        for (int I = 0; I < NB; ++I) v[I] = row[16 * I + c];
        if (jr) v[NB - 1] = r;
        __syncthreads();   // the next step rewrites the rows
    }
};

// Entry `first + lane` of the piece starting at kbeg (lanes below BATCH; past the end: the
// invalid gather word and rating 0).
template <int BATCH, class G>
__device__ __forceinline__ typename G::Entry load_entry(const G& gat,
                                                        const int32_t* __restrict__ colidx,
                                                        const float* __restrict__ vals,
                                                        int64_t kbeg, int64_t total,
                                                        int64_t first, int lane) {
    const bool valid = lane < BATCH && first + lane < total;
    int col = 0;
    float rv = 0.f;
    if (valid) {
        col = colidx[kbeg + first + lane];
        rv = vals[kbeg + first + lane];
    }
    return typename G::Entry{gat.word(col, valid), rv};
}

// The first two index batches of a row piece, loaded ahead of time into registers.
template <class G>
struct RowIndex {
    typename G::Entry q0, q1;
};

// The gather pipeline's in-flight state: operand values and ratings of the steps in flight
// (b[0..kDepth-1] at the top of a group; b[kDepth] is the extra buffer of the rotation).
template <int NBUF>
struct Inflight {
    float b[kGroup][NBUF];
    float r[kGroup];
};

template <class G>
__device__ __forceinline__ void gram_prefetch(const G& gat, const int32_t* __restrict__ colidx,
                                              const float* __restrict__ vals, int64_t kbeg,
                                              int64_t kend, int lane, RowIndex<G>& ix) {
    ix.q0 = load_entry<kBatch>(gat, colidx, vals, kbeg, kend - kbeg, 0, lane);
    ix.q1 = load_entry<kBatch>(gat, colidx, vals, kbeg, kend - kbeg, kBatch, lane);
}

// Put a piece's first two batches into ring slots 0 and 1 (the ring must be idle) and issue
// the gathers of its first kDepth steps.
template <class G>
__device__ __forceinline__ void gram_stage(const G& gat, const RowIndex<G>& ix,
                                           typename G::Entry* ring, int lane,
                                           Inflight<G::kBuf>& in) {
    const int g = lane >> 4;
    if (lane < kBatch) {
        ring[lane] = ix.q0;
        ring[kBatch + lane] = ix.q1;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kDepth; ++j) {
        const typename G::Entry q = ring[4 * j + g];
        in.r[j] = q.r;
        gat.issue(q.e, in.b[j]);
    }
}

// Sub-steps J..kGroup-1 of a group: run step s0 + J from buffer J (a step past the piece's end
// adds nothing) after issuing step s0 + J + kDepth into buffer (J + kDepth) mod kGroup (free: its
// step ran at sub-step J - 1).
template <int J, class G, class Body>
__device__ __forceinline__ void pipe_substeps(const G& gat, const typename G::Entry* ring, int rq,
                                              int s0, int total, int g, Inflight<G::kBuf>& in,
                                              Body& body) {
    if constexpr (J < kGroup) {
        constexpr int JN = (J + kDepth) % kGroup;
        body.take(in.b[J], in.r[J], 4 * (s0 + J) + g < total);
        __builtin_amdgcn_sched_barrier(0);
        int pos = rq + 4 * J;
        if (pos >= kRing) pos -= kRing;
        const typename G::Entry e = ring[pos + g];
        in.r[JN] = e.r;
        gat.issue(e.e, in.b[JN]);
        body.template run<J>();
        pipe_substeps<J + 1>(gat, ring, rq, s0, total, g, in, body);
    }
}

// Run entries [kbeg, kend) of one row piece through the gather pipeline, starting from the state
// gram_stage left in the ring and in `in`.  Per step the body takes the step's operands
// (body.take(B, r, ok): B the loaded values, r the rating, ok whether the step's entry lies in the
// piece), then -- after the gather kDepth steps ahead has been issued -- runs the step
// (body.run<J>(), J the step's place in its group of kGroup; the loop always runs whole groups:
// stopping inside the last group costs more, as a branch per step or as a second copy of the
// group, than the steps of zeros it would skip).
// ring: this wave's LDS ring of kRing entries.  Returns with the ring idle.
template <class G, class Body>
__device__ __forceinline__ void pipe_loop(const G& gat, const int32_t* __restrict__ colidx,
                                          const float* __restrict__ vals, int64_t kbeg,
                                          int64_t kend, typename G::Entry* ring, int lane,
                                          Inflight<G::kBuf>& in, Body& body) {
    const int g = lane >> 4;
    // a row has fewer than 2^31 entries (its columns are distinct int32 indices)
    const int total = (int)(kend - kbeg);
    const int nsteps = (total + 3) >> 2;
    const int ngroups = (nsteps + kGroup - 1) / kGroup;
    typename G::Entry nq{};
    int qb = 0, k = 0;       // group's position in its batch; batch of the group's steps
    int rq = 4 * kDepth;     // ring position of the first step issued in the group
    for (int q = 0; q < ngroups; ++q) {
        // batch k+1 goes into the ring at the top of group 1, one group after its load was
        // issued at the top of group 0 (the store comes first in program order, so its wait
        // never covers the gathers issued after the load)
        if (qb == 1 && k > 0) {
            if (lane < kBatch) ring[((k + 1) & 1) * kBatch + lane] = nq;
            __syncthreads();
        }
        if (qb == 0 && k > 0)
            nq = load_entry<kBatch>(gat, colidx, vals, kbeg, total, (int64_t)(k + 1) * kBatch, lane);
        pipe_substeps<0>(gat, ring, rq, q * kGroup, total, g, in, body);
        rq += 4 * kGroup;
        if (rq >= kRing) rq -= kRing;
        if (++qb == kBatchGroups) {
            qb = 0;
            ++k;
        }
    }
    __syncthreads();   // the ring is refilled by the next piece
}

// ---- the Gram: three-way split bf16 products
//
// The Gram's products run on the bf16 matrix units with every fp32 value split exactly into three
// bf16 parts, x = h + m + l (h: the upper 16 bits of x; m, l: the rest rounded to nearest, twice; 8
// significant bits each), and six of the nine part products kept: hh, hm, mh, mm, hl, lh.  The
// dropped ml and lm reach 2^-23 of hh each, 2^-22 together (2.4e-8 as a root mean square over
// random values), and have one sign for equal values.  Part products are exact in fp32.  A group of 32
// entries is one K = 32 step: its products start from zero, smallest parts first, and their sum is
// added to the fp32 accumulator once, so that an accumulator is rounded once per 32 entries (the fp32
// v_mfma_f32_16x16x4_f32 rounds it for every entry).  The sums' error against fp64, relative, as a root
// mean square, beside one FMA per entry: 3.0e-8 (4.5e-8) for 8 random entries, 2.6e-8 (8.4e-8) for 32,
// 4.0e-8 (1.7e-7) for 128; for as many equal entries 3.9e-8 (5.3e-8), 3.7e-8 (2.3e-7), 3.9e-8 (9.5e-7).  Only the shortest sums
// lose: 4.3e-8 (2.5e-8) for one entry.  So a piece of at most kPlainEntries = 16 entries, up to which
// the dropped products may also exceed the FMAs' largest error, takes fp32 products instead: before
// its group runs, from the same gathered values, and the group then runs with parts of zero (a
// group of its own would cost registers that f = 80 to 112 do not have: spills, movie user side
// 9.9 -> 10.7 ms, 1/32 of the wiki one 21.1 -> 23.5).  Rows of 5 ratings on average pay 2-6% for it, the
// wiki part (62) 0.9%, the movie sides nothing.
//
// Why: v_mfma_f32_16x16x4_f32 takes 32 cycles for 4 entries of a tile, 256 cycles for 32, and
// nothing else runs on the SIMD meanwhile (fp32 MFMA and VALU work exclude each other).  Six
// v_mfma_f32_16x16x32_bf16 take 96, and the other wave's VALU work runs beside them.
//
// The gather layout is unchanged: lane (g, c) loads column 16 I + c of entry 4 j + g for step j of
// the group's eight, and holds, after the split, K slots 8 g + j of its column, which is the bf16
// operand layout (K slot order is the same for both operands, so any order serves).
//
// Registers bound the design (two waves per SIMD, 256 each, for f < 116): 4 per tile for the
// accumulators, 12 per block for the parts and 8 per block for the gathered values do not fit
// together at f = 100.  So the columns of tiles are run last first, column J taking the tiles (I, J),
// I <= J; after it the parts of block J are dead, and their registers take the next group's
// gathers.  (Splitting the next group's block J beside column J - 1 instead, each block gathered three
// columns ahead, measured slower: 10.8 against 10.2 ms on the movie user side; the parts then live
// through the solve.)
//
// A packed last block holds, as one operand, the h parts in lanes 0..q-1, the m parts in q..2q-1 and
// the l parts in 2q..3q-1: three products per tile (by the other operand's l, m and h parts)
// instead of six, one for the tile (NB-1, NB-1), and 4 registers instead of 12.  The column groups
// are added when the Gram is complete (fold_packed).
constexpr int kGroupSteps = 8;
constexpr int kGroupEntries = 4 * kGroupSteps;
constexpr int kPlainEntries = 16;              // pieces up to this long take fp32 products
constexpr int kGramBatch = kWave;              // index batch: one entry per lane, two groups
constexpr int kGramRing = 2 * kGramBatch;

typedef unsigned u4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

// How split_pair takes h: the kept bits of a value, and the v_perm selector of two values' upper halves.
// With kNothing all three parts are zero (for finite values).
struct Cut {
    unsigned bits, pick;
};
constexpr Cut kUpperHalf{0xFFFF0000u, 0x07060302u}, kNothing{0xFFFFFFFFu, 0x0C0C0C0Cu};

// The three parts of x and y, packed (x in the low half).  h is cut, not rounded, so that no
// finite value's parts overflow.
__device__ __forceinline__ void split_pair(float x, float y, const Cut& cut, unsigned& h, unsigned& m,
                                           unsigned& l) {
    const unsigned xb = __builtin_bit_cast(unsigned, x), yb = __builtin_bit_cast(unsigned, y);
    h = __builtin_amdgcn_perm(yb, xb, cut.pick);
    const float rx = x - __builtin_bit_cast(float, xb & cut.bits);
    const float ry = y - __builtin_bit_cast(float, yb & cut.bits);
    m = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{rx, ry}, bf2));
    const float sx = rx - __builtin_bit_cast(float, m << 16);
    const float sy = ry - __builtin_bit_cast(float, m & 0xFFFF0000u);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector(f2{sx, sy}, bf2));
}

__device__ __forceinline__ f4 mfma_bf16(u4 a, u4 b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8, a),
                                                   __builtin_bit_cast(bf8, b), c, 0, 0, 0);
}

// The parts of a group's operands: element p of a part holds steps 2p and 2p + 1.
template <int NB, int LAST>
struct Parts {
    static constexpr int kFull = LAST == kLastTiles ? NB : NB - 1;   // blocks with three parts
    u4 h[kFull], m[kFull], l[kFull];
    u4 last;   // kLastPacked: the last block
};

// Tiles that the products fill, and the registers of a group's accumulators and parts.
constexpr int gram_tiles(int nb, int last) { return ntiles(last == kLastRating ? nb - 1 : nb); }
constexpr int gram_registers(int nb, int last) {
    return 4 * gram_tiles(nb, last) + 12 * (last == kLastTiles ? nb : nb - 1) +
           (last == kLastPacked ? 4 : 0) + (last == kLastRating ? nb - 1 : 0);
}
// f = 113 to 127 take fp32 products throughout, in half groups of 16 entries: with the parts beside 144
// accumulator registers only one wave per SIMD fits, and nothing runs beside its solve.  2M ratings of
// 400,000 users at f = 113 and 120: 8.65 and 8.47 ms with parts, 6.81 and 6.54 so; 20M of 200,000
// users 6.05 and 6.03, 6.18 and 5.94.  (The products of every four entries straight into the
// accumulators: 6.62, 6.45, 5.88 and 5.73, but an error against fp64 of 2.7e-6 instead of 1.5e-6 on
// the longer rows.)  f = 112 fits two waves with its parts: 4.1 ms, with one wave 5.7.
constexpr bool gram_fp32(int nb, int last) { return nb == 8 && last != kLastRating; }
// The least waves per SIMD that the compiler is held to: two where accumulators and parts leave 50
// registers of 256 for the rest, and what f = 16, 32 and 48 take without spilling (the 64-bit parts
// form, whose waves bound the others', would take 102 and 130 registers at f = 16 and 32 and lose one
// of five and of four waves: 361 against 327 us on 20M ratings of 200,000 users at f = 16, 659 against
// 573 at f = 32).
constexpr int gram_waves(int nb, int last) {
    if (gram_fp32(nb, last)) return 2;
    if (nb <= 4 && last == kLastRating) return 7 - nb;
    return gram_registers(nb, last) <= 206 ? 2 : 1;
}

// The gathered values of a group, step by step.
template <class G>
struct Raw {
    float b[kGroupSteps][G::kBuf];
};

// Issue the gathers of steps [J0, J1) of the group whose entries start at `ring`.
template <int J0, int J1, class G>
__device__ __forceinline__ void issue_steps(const G& gat, const typename G::Entry* ring, int g,
                                            Raw<G>& raw) {
#pragma unroll
    for (int j = J0; j < J1; ++j) gat.issue(ring[4 * j + g].e, raw.b[j]);
}

// Steps of the next group that may have been issued before column J is run (J = -1: when all are
// done): as many as the registers left over and the parts of the finished blocks allow.  (A budget
// of 190 or 200 registers instead of 184 spills: movie user side 10.33 and 10.43 against 9.89 ms;
// 160 reads the same there and 22% slower with the 64-bit gather.)
template <int NB, int LAST>
constexpr int steps_before(int J) {
    constexpr int top = LAST == kLastRating ? NB - 2 : NB - 1;
    constexpr int per_step = LAST == kLastRating ? NB - 1 : NB;
    if (J < 0 || gram_waves(NB, LAST) == 1) return kGroupSteps;
    int freed = 184 - gram_registers(NB, LAST);
    for (int k = top; k > J; --k) freed += LAST == kLastPacked && k == NB - 1 ? 4 : 12;
    const int steps = freed <= 0 ? 0 : freed / per_step;
    return steps > kGroupSteps ? kGroupSteps : steps;
}

template <int NB, int LAST, int J, class G>
__device__ __forceinline__ void tile_columns(const Parts<NB, LAST>& a, f4 (&acc)[ntiles(NB)],
                                             const G& gat, const typename G::Entry* next, int g,
                                             Raw<G>& raw) {
    constexpr f4 zero = f4{0.f, 0.f, 0.f, 0.f};
    constexpr bool packed = LAST == kLastPacked && J == NB - 1;
#pragma unroll
    for (int I0 = 0; I0 <= J; I0 += 2) {   // two chains side by side
        f4 t[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int I = I0 + i;
            if (I > J) continue;
            if constexpr (packed) {
                if (I == J) {
                    t[i] = mfma_bf16(a.last, a.last, zero);
                } else {
                    t[i] = mfma_bf16(a.l[I], a.last, zero);
                    t[i] = mfma_bf16(a.m[I], a.last, t[i]);
                    t[i] = mfma_bf16(a.h[I], a.last, t[i]);
                }
            } else {
                t[i] = mfma_bf16(a.l[I], a.h[J], zero);
                t[i] = mfma_bf16(a.h[I], a.l[J], t[i]);
                t[i] = mfma_bf16(a.m[I], a.m[J], t[i]);
                t[i] = mfma_bf16(a.m[I], a.h[J], t[i]);
                t[i] = mfma_bf16(a.h[I], a.m[J], t[i]);
                t[i] = mfma_bf16(a.h[I], a.h[J], t[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (I0 + i <= J) acc[tu(NB, I0 + i, J)] += t[i];
    }
    __builtin_amdgcn_sched_barrier(0);
    issue_steps<steps_before<NB, LAST>(J), steps_before<NB, LAST>(J - 1)>(gat, next, g, raw);
    if constexpr (J > 0) tile_columns<NB, LAST, J - 1>(a, acc, gat, next, g, raw);
}

// A row piece longer than a part (kPart entries by default; a power of two times a group's 32 entries)
// runs in parts (the last one shorter): each part's Gram is accumulated in
// registers from zero, and the parts' sums are added in order into the wave's own
// partial-accumulator slot in the workspace, the second level of a two-level sum, so that no fp32
// running sum spans more than a part (a column of tens of millions of ratings otherwise
// accumulates over a million entries in one register chain).  After the last part the slot is
// added into the registers and the piece goes on as one accumulator.
constexpr int64_t kPart = 1 << 16;

// A partial-accumulator slot: tile t of lane l at f4 index 64 t + l (16 contiguous bytes per
// lane, 1 KiB per tile).
template <int NB>
__device__ __forceinline__ void store_slot(const f4 (&acc)[ntiles(NB)], float* __restrict__ slot,
                                           int lane) {
    f4* s = reinterpret_cast<f4*>(slot);
#pragma unroll
    for (int t = 0; t < ntiles(NB); ++t) s[t * kWave + lane] = acc[t];
}

// acc += slot.  All loads are issued before the first add (a dependent load-add chain would
// leave one load in flight at a time).
template <int NB>
__device__ __forceinline__ void add_slot(f4 (&acc)[ntiles(NB)], const float* __restrict__ slot,
                                         int lane) {
    const f4* s = reinterpret_cast<const f4*>(slot);
    f4 v[ntiles(NB)];
#pragma unroll
    for (int t = 0; t < ntiles(NB); ++t) v[t] = s[t * kWave + lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < ntiles(NB); ++t) acc[t] += v[t];
}

// slot += acc, four tiles at a time (the temporaries stay at 16 registers beside the
// accumulators).
template <int NB>
__device__ __forceinline__ void fold_into_slot(const f4 (&acc)[ntiles(NB)],
                                               float* __restrict__ slot, int lane) {
    f4* s = reinterpret_cast<f4*>(slot);
#pragma unroll
    for (int t0 = 0; t0 < ntiles(NB); t0 += 4) {
        f4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t0 + j < ntiles(NB)) v[j] = s[(t0 + j) * kWave + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t0 + j < ntiles(NB)) s[(t0 + j) * kWave + lane] = v[j] + acc[t0 + j];
        __builtin_amdgcn_sched_barrier(0);
    }
}

// acc += slot, four tiles at a time.
template <int NB>
__device__ __forceinline__ void add_slot_in_fours(f4 (&acc)[ntiles(NB)],
                                                  const float* __restrict__ slot, int lane) {
    const f4* s = reinterpret_cast<const f4*>(slot);
#pragma unroll
    for (int t0 = 0; t0 < ntiles(NB); t0 += 4) {
        f4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t0 + j < ntiles(NB)) v[j] = s[(t0 + j) * kWave + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (t0 + j < ntiles(NB)) acc[t0 + j] += v[j];
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The column groups of a packed last block (parts h, m, l) into its real columns 0..q-1, the row
// groups of the tile (NB-1, NB-1) into its real rows, the rest of the tiles zero.
// scratch: NB KiB of LDS, 16-byte aligned.
template <int NB>
__device__ __forceinline__ void fold_packed(f4 (&acc)[ntiles(NB)], int q, void* scratch,
                                            int lane) {
    const int g = lane >> 4, c = lane & 15;
    f4* sc = reinterpret_cast<f4*>(scratch);
#pragma unroll
    for (int I = 0; I < NB; ++I) sc[I * kWave + lane] = acc[tu(NB, I, NB - 1)];
    __syncthreads();
#pragma unroll
    for (int I = 0; I < NB; ++I) {
        f4 v = f4{0.f, 0.f, 0.f, 0.f};
        if (c < q) {
            const f4* p = sc + I * kWave + lane;
            v = (p[2 * q] + p[q]) + p[0];
        }
        acc[tu(NB, I, NB - 1)] = v;
    }
    __syncthreads();
    // row i of the last tile is element i & 3 of lane (i / 4, c): float 64 (i / 4) + 4 c + (i & 3)
    float* s = reinterpret_cast<float*>(scratch);
    *reinterpret_cast<f4*>(s + 4 * lane) = acc[tu(NB, NB - 1, NB - 1)];
    __syncthreads();
    f4 v = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = 4 * g + r;
        if (i < q && c < q) {
            const auto at = [&](int row) { return s[64 * (row >> 2) + 4 * c + (row & 3)]; };
            v[r] = (at(i + 2 * q) + at(i + q)) + at(i);
        }
    }
    acc[tu(NB, NB - 1, NB - 1)] = v;
    __syncthreads();
}

// The rating column's sums (b[I] at lane (e, c): entry slot e's part of M[16 I + c][f]) into column
// 0 of the last block column's tiles, the rest of those zero.
template <int NB>
__device__ __forceinline__ void fold_rating(f4 (&acc)[ntiles(NB)], const float (&b)[NB - 1],
                                            void* scratch, int lane) {
    const int g = lane >> 4, c = lane & 15;
    float* sb = reinterpret_cast<float*>(scratch);
#pragma unroll
    for (int I = 0; I < NB - 1; ++I) sb[I * kWave + lane] = b[I];
    __syncthreads();
#pragma unroll
    for (int I = 0; I < NB; ++I) {
        f4 v = f4{0.f, 0.f, 0.f, 0.f};
        if (I < NB - 1 && c == 0) {
            const f4* s = reinterpret_cast<const f4*>(sb + I * kWave + 4 * g);   // slot e: s[4e]
            v = ((s[0] + s[4]) + s[8]) + s[12];
        }
        acc[tu(NB, I, NB - 1)] = v;
    }
    __syncthreads();
}

template <int NB, int LAST, class G, bool PARTS>
struct GramBody {
    static constexpr bool kFp32 = gram_fp32(NB, LAST);
    static constexpr bool kParts = PARTS, kPlain = !kFp32;
    static constexpr int kTop = LAST == kLastRating ? NB - 2 : NB - 1;   // last column of products
    int part_mask;        // groups per part - 1 (a power of two - 1)
    const G& gat;
    f4 (&acc)[ntiles(NB)];
    int q;                // real columns of the last block
    int third;            // kLastPacked: the part of the last block this lane holds (0: h, 1: m, 2: l)
    void* scratch;        // LDS for fold_packed and fold_rating
    float* wslot;         // the wave's slot
    int lane;
    const typename G::Entry* cur = nullptr;   // kFp32: the group's entries
    Cut cut = kUpperHalf; // kNothing: the piece's products are in acc already (plain)
    float b[NB > 1 ? NB - 1 : 1];   // kLastRating: the rating column's sums
    Parts<NB, LAST> a;
    // the accumulators from zero (those of the last block column are set by finish where no
    // products fill them)
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int I = 0; I <= kTop; ++I)
#pragma unroll
            for (int J = I; J <= kTop; ++J) acc[tu(NB, I, J)] = f4{0.f, 0.f, 0.f, 0.f};
        if constexpr (LAST == kLastRating) {
#pragma unroll
            for (int I = 0; I < NB - 1; ++I) b[I] = 0.f;
        }
    }
    // the products of a piece of at most 4 kSteps entries in fp32, four entries a step, into the
    // accumulators (the rating column of kLastRating is take's)
    template <int kSteps>
    __device__ __forceinline__ void plain(const Raw<G>& raw, const typename G::Entry* ring, int g) {
        float x[kSteps][G::kBlocks];
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const float r = ring[4 * j + g].r;
            gat.operands(raw.b[j], r, x[j]);
            // a packed last block's copies of its columns add nothing
            if constexpr (LAST == kLastPacked) x[j][NB - 1] = third == 0 ? x[j][NB - 1] : 0.f;
        }
#pragma unroll
        for (int I = 0; I <= kTop; ++I)
#pragma unroll
            for (int J = I; J <= kTop; ++J) {
                f4 t = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < kSteps; ++j)
                    t = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][I], x[j][J], t, 0, 0, 0);
                acc[tu(NB, I, J)] = t;
            }
    }
    // the group's operands from its gathered values and its ratings (in the ring)
    __device__ __forceinline__ void take(const Raw<G>& raw, const typename G::Entry* ring) {
        if constexpr (kFp32) {
            cur = ring;
            return;
        }
        const int g = lane >> 4;
#pragma unroll
        for (int p = 0; p < kGroupSteps / 2; ++p) {
            float x[G::kBlocks], y[G::kBlocks];
            const float rx = ring[4 * (2 * p) + g].r, ry = ring[4 * (2 * p + 1) + g].r;
            gat.operands(raw.b[2 * p], rx, x);
            gat.operands(raw.b[2 * p + 1], ry, y);
#pragma unroll
            for (int I = 0; I < G::kBlocks; ++I) {
                unsigned h, m, l;
                split_pair(x[I], y[I], cut, h, m, l);
                if constexpr (LAST == kLastRating)
                    b[I] = __builtin_fmaf(y[I], ry, __builtin_fmaf(x[I], rx, b[I]));
                if (LAST == kLastPacked && I == NB - 1) {
                    a.last[p] = third == 0 ? h : (third == 1 ? m : l);
                } else {
                    a.h[I][p] = h;
                    a.m[I][p] = m;
                    a.l[I][p] = l;
                }
            }
        }
    }
    __device__ __forceinline__ void run(const typename G::Entry* next, Raw<G>& raw) {
        if constexpr (kFp32) {
            const int g = lane >> 4;
            constexpr int kHalf = kGroupSteps / 2;
#pragma unroll
            for (int j0 = 0; j0 < kGroupSteps; j0 += kHalf) {
                float x[kHalf][G::kBlocks];
#pragma unroll
                for (int j = 0; j < kHalf; ++j) {
                    gat.operands(raw.b[j0 + j], cur[4 * (j0 + j) + g].r, x[j]);
                    if constexpr (LAST == kLastPacked) x[j][NB - 1] = third == 0 ? x[j][NB - 1] : 0.f;
                }
#pragma unroll
                for (int I = 0; I <= kTop; ++I)
#pragma unroll
                    for (int J = I; J <= kTop; ++J) {
                        f4 t = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int j = 0; j < kHalf; ++j)
                            t = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][I], x[j][J], t, 0, 0, 0);
                        acc[tu(NB, I, J)] += t;
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = j0; j < j0 + kHalf; ++j) gat.issue(next[4 * j + g].e, raw.b[j]);
            }
            return;
        }
        issue_steps<0, steps_before<NB, LAST>(kTop)>(gat, next, lane >> 4, raw);
        tile_columns<NB, LAST, kTop>(a, acc, gat, next, lane >> 4, raw);
    }
    __device__ __forceinline__ void finish() {
        if constexpr (LAST == kLastPacked) fold_packed<NB>(acc, q, scratch, lane);
        if constexpr (LAST == kLastRating) fold_rating<NB>(acc, b, scratch, lane);
    }
    // at a part boundary the accumulators so far are stored into, or added to, the wave's slot,
    // and start again from zero
    __device__ __forceinline__ void flush(bool first) {
        finish();
        if (first) store_slot<NB>(acc, wslot, lane);
        else fold_into_slot<NB>(acc, wslot, lane);
        clear();
    }
};

// The lane, computed on the spot: an address made from it is not kept in a register across the loop, or
// spilled and loaded again, which waits for every gather in flight (the parts form at f = 100 did so
// once per 64 entries).
__device__ __forceinline__ int fresh_lane() {
    unsigned zero = 0;
    asm volatile("" : "+s"(zero));
    return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
}

// The first batch of a piece into ring slot `slot`, and the gathers of its first group.
template <class G>
__device__ __forceinline__ void start_piece(const G& gat, const typename G::Entry& first,
                                            typename G::Entry* ring, int slot, int lane,
                                            Raw<G>& raw) {
    ring[slot * kGramBatch + lane] = first;
    __syncthreads();
    issue_steps<0, kGroupSteps>(gat, ring + slot * kGramBatch, lane >> 4, raw);
}

// Run entries [kbeg, kend) of one row piece, whose first group's gathers are in flight, group by
// group: the body takes the group's operands (take), then runs its products while the next
// group's gathers are issued (run).  After the last group those are the next piece's (its first
// batch, next_first, goes into the ring; without a next piece the last group is gathered once
// more and not used).  The index batches alternate between the ring's two slots; `slot` is the slot
// of the piece's first batch, and of the next piece's on return.  Batch k + 1 is loaded (one entry
// per lane) at batch k's first group and stored at its second, whose run reads it first.
template <class G, class Body>
__device__ __forceinline__ void group_loop(const G& gat, const int32_t* __restrict__ colidx,
                                           const float* __restrict__ vals, int64_t kbeg,
                                           int64_t kend, typename G::Entry* ring, int& slot,
                                           int lane, Raw<G>& raw, bool more,
                                           const typename G::Entry& next_first, Body& body) {
    // a row has fewer than 2^31 entries (its columns are distinct int32 indices)
    const int total = (int)(kend - kbeg);
    const int ngroups = (total + kGroupEntries - 1) / kGroupEntries;
    if constexpr (Body::kPlain) {
        if (total <= kPlainEntries) {
            const int l = fresh_lane();
            const typename G::Entry* cur = ring + slot * kGramBatch;
            if (total <= kPlainEntries / 2) body.template plain<kPlainEntries / 8>(raw, cur, l >> 4);
            else body.template plain<kPlainEntries / 4>(raw, cur, l >> 4);
            body.cut = kNothing;
        }
    }
    typename G::Entry nq{};
    for (int q = 0; q < ngroups; ++q) {
        if constexpr (Body::kParts) {
            if (q > 0 && (q & body.part_mask) == 0) body.flush(q == body.part_mask + 1);
        }
        const int other = slot ^ 1;   // `slot` holds this group's batch
        const int odd = q & 1;
        const typename G::Entry* cur = ring + slot * kGramBatch + odd * kGroupEntries;
        const bool last = q + 1 == ngroups;
        if (!odd && !last)
            nq = load_entry<kGramBatch>(gat, colidx, vals, kbeg, total,
                                        (int64_t)(q / 2 + 1) * kGramBatch, lane);
        body.take(raw, cur);
        const typename G::Entry* next = odd ? cur : cur + kGroupEntries;
        if (last) next = cur;
        if (last ? more : odd) {
            // (by members: a choice between the objects is one between addresses, and keeps both in
            // private memory)
            ring[other * kGramBatch + fresh_lane()] =
                typename G::Entry{last ? next_first.e : nq.e, last ? next_first.r : nq.r};
            __syncthreads();
            next = ring + other * kGramBatch;
        }
        body.run(next, raw);
        if (last || odd) slot = other;
    }
}

// The gather stage made visible (test and debug support): for one row, the values the Gram's
// operands are split from -- the same Gather form, index ring and group loop as k_herm_solve -- are
// written out per entry instead of multiplied.  Entry k's record has 16 (NB + 3) floats: block I
// of the operand at 16 I + c (lane c of the entry's 16-lane group, zero in the second and third
// copies of a packed block's columns; the rating where the rating column has no block); for f mod 16 =
// 0 or 4, unless the last block is an ordinary one, its columns by quads, lane c holding column c & 3
// of the quad, at 16 (NB + p) + c (untouched otherwise); and the rating at 16 (NB + 2) + c.
template <int NB>
constexpr int dump_floats() { return 16 * (NB + 3); }

template <int NB, int LAST, class G>
struct DumpBody {
    static constexpr bool kParts = false, kPlain = false;
    const G& gat;
    float* __restrict__ out;
    int64_t limit;   // entries that fit in out
    int q, total, lane, group;
    __device__ __forceinline__ void take(const Raw<G>& raw, const typename G::Entry* ring) {
        const int g = lane >> 4, c = lane & 15;
#pragma unroll
        for (int j = 0; j < kGroupSteps; ++j) {
            const float r = ring[4 * j + g].r;
            float v[G::kBlocks];
            gat.operands(raw.b[j], r, v);
            const float quad = __shfl(v[G::kBlocks - 1], (lane & 48) | (c & 3));
            const int64_t k = (int64_t)kGroupEntries * group + 4 * j + g;
            if (k < total && k < limit) {
                float* rec = out + k * dump_floats<NB>();
#pragma unroll
                for (int I = 0; I < NB - 1; ++I) rec[16 * I + c] = v[I];
                if constexpr (LAST == kLastRating) rec[16 * (NB - 1) + c] = c == 0 ? r : 0.f;
                else rec[16 * (NB - 1) + c] = LAST == kLastTiles || c < q ? v[NB - 1] : 0.f;
                if (LAST == kLastPacked && q == 5) rec[16 * NB + c] = quad;
                if (LAST == kLastRating || (LAST == kLastPacked && q == 5))
                    rec[16 * (NB + q / 4) + c] = (c & 3) == 0 ? r : 0.f;
                rec[16 * (NB + 2) + c] = r;
            }
        }
        ++group;
    }
    __device__ __forceinline__ void run(const typename G::Entry* next, Raw<G>& raw) {
        issue_steps<0, kGroupSteps>(gat, next, lane >> 4, raw);
    }
};

template <int NB, int BUF, int LAST>
__global__ __launch_bounds__(kWave) void k_gather_dump(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ vals, const float* __restrict__ theta, int64_t n, int f, int64_t u,
    float* __restrict__ out, int64_t limit) {
    using G = Gather<NB, BUF, LAST>;
    __shared__ typename G::Entry ring[kGramRing];
    __shared__ __attribute__((aligned(16))) float stage[BUF == kFormStaged ? stage_floats(NB) : 4];
    const int lane = threadIdx.x;
    if constexpr (BUF == kFormStaged) {
        for (int i = lane; i < stage_floats(NB); i += kWave) stage[i] = 0.f;
        __syncthreads();
    }
    const G gat(theta, n, f, lane & 15, stage);
    const int64_t kbeg = rowptr[u], kend = rowptr[u + 1];
    if (kbeg == kend) return;
    const typename G::Entry first =
        load_entry<kGramBatch>(gat, colidx, vals, kbeg, kend - kbeg, 0, lane);
    Raw<G> raw;
    int slot = 0;
    start_piece(gat, first, ring, slot, lane, raw);
    DumpBody<NB, LAST, G> body{gat, out, limit, f - 16 * (NB - 1) + 1, (int)(kend - kbeg), lane, 0};
    group_loop(gat, colidx, vals, kbeg, kend, ring, slot, lane, raw, false, first, body);
}

// ------------------------------------------------------------------ solve in registers ---

// LDS scratch of one wave for the solve.
template <int NB>
struct SolveLds {
    float W[NB][256];   // -W_K = -L_KK^{-1} per block, column-major: W[K][16 j + i] = -W_K[i][j]
    float T[256];       // a diagonal tile, row-major
    float y[16 * NB];   // forward-substitution result (row f of the augmented factor)
    float x[16 * NB];   // solution, zero past f
    float z[16];
};

// Registers of factor_tile (see there).
struct FactorRegs {
    float tr[4], wr[4], to[4], wo[4];   // to/wo[0] unused
};

// Pivot kk = 4 B + P of factor_tile.  The next pivot waits on this one's readlane, s, s^2, the
// product for the next row and that row's update, so the next row (P + 1) is updated first.
// One transcendental per pivot (s = piv^{-1/2}; 1/piv = s^2).
template <int B, int P, bool kFull>
__device__ __forceinline__ void factor_pivot(FactorRegs& R, bool live, int& pmin, int& pmax,
                                             float* ystore) {
    constexpr int kk = 4 * B + P;
    // the pivot T[kk][kk] = -N[kk][kk]: lane kk's value with the sign bit flipped (scalar)
    int pb = __builtin_amdgcn_readlane(__builtin_bit_cast(int, R.tr[P]), kk) ^ 0x80000000;
    pb = live ? pb : 0x3F800000;   // 1.0f
    pmin = min(pmin, pb);
    pmax = max(pmax, pb);
    asm volatile("" : "+s"(pmin), "+s"(pmax));   // fold in now, in scalar registers
    const float s = live ? __builtin_amdgcn_rsqf(__builtin_bit_cast(float, pb)) : 0.f;
    const float s2 = s * s;   // 1 / piv
    const float at = s2 * R.tr[P];          // N[kk][c] / piv
    const float aw = s2 * R.wr[P];          // (-W)[kk][c] / piv
    if (ystore) ystore[kk] = -s * R.tr[P];  // L[nlast][kk] = s T[kk][nlast]
    R.wr[P] *= s;                           // row kk of -W is final
    // Order: row P + 1 (W, then T: the W update reads T's column kk before the T update changes
    // it), then the other rows' W updates, then their T updates.  A DPP read of a T register then
    // sits at least n - 1 instructions after the previous pivot's write of it (n row updates
    // here); a block's first pivot always waits (its sources were loaded or carried over the
    // block's branch).
    // (without the later rows, kFull = false, every pivot waits)
    constexpr int n = (3 - P) + (3 - B);
    if constexpr (P == 0 || n < 3 || !kFull) dpp_settle();
    if constexpr (P < 3) {
        R.wr[P + 1] = fmac_bcast<kk>(R.wr[P + 1], R.tr[P + 1], aw);
        R.tr[P + 1] = fmac_bcast<kk>(R.tr[P + 1], R.tr[P + 1], at);
    }
#pragma unroll
    for (int j = P + 2; j < 4; ++j) R.wr[j] = fmac_bcast<kk>(R.wr[j], R.tr[j], aw);
    if constexpr (kFull) {
#pragma unroll
        for (int bb = B + 1; bb < 4; ++bb) R.wo[bb] = fmac_bcast<kk>(R.wo[bb], R.to[bb], aw);
    }
#pragma unroll
    for (int j = P + 2; j < 4; ++j) R.tr[j] = fmac_bcast<kk>(R.tr[j], R.tr[j], at);
    if constexpr (kFull) {
#pragma unroll
        for (int bb = B + 1; bb < 4; ++bb) R.to[bb] = fmac_bcast<kk>(R.to[bb], R.to[bb], at);
    }
}

// Factor and invert the symmetric 16 x 16 diagonal tile T, staged negated in S.T (row-major:
// N = -T, as the accumulator tiles hold it), right-looking: pivot kk = T[kk][kk] scales row kk of
// W = L_KK^{-1} (built from the identity) by s = piv^{-1/2} and then takes
// T[i][c] -= T[i][kk] T[kk][c] / piv and W[i][c] -= T[i][kk] W[kk][c] / piv for every later row i.
// The registers hold N and -W, for which the same steps read N[i][c] += N[i][kk] N[kk][c] / piv
// and (-W)[i][c] += N[i][kk] (-W)[kk][c] / piv; -W goes to S.W, as the panel and the back
// substitution use it.  Lane (g, c) holds column c.  The rows of the current 4-row block b sit in every group
// (tr, wr: rows 4b + j); a later row 4b' + g is held by group g alone (to, wo[b']), so each
// group updates a quarter of them.  Either way the multiplier T[i][kk] is the row's own register
// in lane kk (DPP row_newbcast:kk), and N[kk][c] / piv, (-W)[kk][c] / piv are the lane's own (the
// current block is replicated).  Between blocks the groups trade the next block's rows through
// LDS.  Columns left of the pivot are not needed again; they go to zero as the elimination
// proceeds instead of being masked.  npiv real pivots: a block with none is skipped (last block
// only) and a pivot past npiv inside a block runs with s = 0, so it adds nothing (a branch per
// pivot would make the register allocator copy DPP sources right before their reads); rows of W
// past npiv stay as the updates left them (the identity in the padding, zero for a pivot skipped
// inside a block).  In the last block the row nlast is the augmented b row, whose L entries are y
// (written to S.y).  pmin/pmax track the pivots' bit patterns: every pivot was positive and
// finite (not NaN, not +inf) iff pmin > 0 and pmax < the bits of +inf.
// kFull = false: the tile has at most 4 real rows (the last block when f - 16 (NB - 1) <= 4).
// Then the rows past the first block are neither pivots nor needed (the b row's L entries come
// from the pivot rows' column nlast), so only block 0 is factored and rows 4..15 of -W are
// written as zeros (the back substitution multiplies them by zeros).
template <int NB, bool kFull, int B = 0>
__device__ __forceinline__ void factor_blocks(SolveLds<NB>& S, FactorRegs& R, int K, int npiv,
                                              float* ystore, int& pmin, int& pmax, int lane) {
    const int g = lane >> 4, c = lane & 15;
    if (4 * B < npiv) {
        factor_pivot<B, 0, kFull>(R, 4 * B + 0 < npiv, pmin, pmax, ystore);
        factor_pivot<B, 1, kFull>(R, 4 * B + 1 < npiv, pmin, pmax, ystore);
        factor_pivot<B, 2, kFull>(R, 4 * B + 2 < npiv, pmin, pmax, ystore);
        factor_pivot<B, 3, kFull>(R, 4 * B + 3 < npiv, pmin, pmax, ystore);
    }
    if constexpr (!kFull) {
        const f4 z = f4{0.f, 0.f, 0.f, 0.f};
        *reinterpret_cast<f4*>(&S.W[K][c * 16 + 4 * g]) =
            g == 0 ? f4{R.wr[0], R.wr[1], R.wr[2], R.wr[3]} : z;
        return;
    }
    if (g == 0)
        *reinterpret_cast<f4*>(&S.W[K][c * 16 + 4 * B]) = f4{R.wr[0], R.wr[1], R.wr[2], R.wr[3]};
    if constexpr (B < 3) {
        // rows 4(B+1) + j: group j's to/wo[B+1] -> every group's tr/wr[j].  The staged tile is
        // in registers now; its LDS holds the exchange.
        float* X = S.T;
        __syncthreads();
        *reinterpret_cast<float2*>(&X[c * 8 + 2 * g]) = float2{R.to[B + 1], R.wo[B + 1]};
        __syncthreads();
        const f4 u0 = *reinterpret_cast<const f4*>(&X[c * 8]);
        const f4 u1 = *reinterpret_cast<const f4*>(&X[c * 8 + 4]);
        R.tr[0] = u0[0]; R.wr[0] = u0[1]; R.tr[1] = u0[2]; R.wr[1] = u0[3];
        R.tr[2] = u1[0]; R.wr[2] = u1[1]; R.tr[3] = u1[2]; R.wr[3] = u1[3];
        factor_blocks<NB, kFull, B + 1>(S, R, K, npiv, ystore, pmin, pmax, lane);
    }
}

template <int NB, bool kFull>
__device__ __forceinline__ void factor_tile(SolveLds<NB>& S, int K, int npiv, int nlast,
                                            int& pmin, int& pmax, int lane) {
    const int g = lane >> 4, c = lane & 15;
    FactorRegs R;
    // No matrix instruction moves past this point, and the first inline FMA comes ten wait states after
    // it, while the tile loads from LDS (the panel's and trailing products may have results still
    // under way, or be reading SrcC registers that are given out again here).
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) R.tr[j] = S.T[c * 16 + j];
    R.to[0] = R.wo[0] = 0.f;
    if constexpr (kFull) {
#pragma unroll
        for (int bb = 1; bb < 4; ++bb) R.to[bb] = S.T[c * 16 + 4 * bb + g];
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 9");
    // -identity: row j in lanes c == j; row 4b' + g in lanes 16 g + 4 b' + g
#pragma unroll
    for (int j = 0; j < 4; ++j) R.wr[j] = in_lanes(0x0001000100010001ull << j) ? -1.f : 0.f;
    if constexpr (kFull) {
#pragma unroll
        for (int bb = 1; bb < 4; ++bb)
            R.wo[bb] = in_lanes(0x0008000400020001ull << (4 * bb)) ? -1.f : 0.f;
    } else {
#pragma unroll
        for (int bb = 1; bb < 4; ++bb) R.to[bb] = R.wo[bb] = 0.f;
    }
    float* ystore = ((K == NB - 1) && lane == nlast) ? &S.y[16 * K] : nullptr;
    factor_blocks<NB, kFull>(S, R, K, npiv, ystore, pmin, pmax, lane);
}

// Block K's acc-indexed steps, one instantiation per K (the block loop runs at run time so the
// factor code above exists once):
// The tiles not yet factored hold the Schur complement negated (-U), so that the trailing update
// is a plain multiply-accumulate.
//   stage: diagonal tile -U_KK = acc, less lambda n_u on its diagonal (real columns only),
//          -> S.T, so that lane c can read row (= column) c;
//   panel: D_I = W_K U_{K,I} = L_IK^T for I > K (stored positive); y_K from the augmented
//          column; trailing update -U_{J,I} += D_J^T D_I for K < J <= I.  Each product is four
//          16x16x4 MFMAs over the permuted contraction index p = 4g + s, under which lane (g, c)
//          element s of a C-layout tile is both the A operand (of its transpose) and the B
//          operand;
//   matvec: sum_{I>K} D_{K,I}[4g + r][c] x[16 I + c] per lane (summed over c by the caller).
template <int NB, int K>
struct Block {
    static __device__ __forceinline__ void stage(const f4 (&acc)[ntiles(NB)], SolveLds<NB>& S,
                                                 float lam_n, int nlast, int lane) {
        const int g = lane >> 4, c = lane & 15;
        f4 t = acc[tu(NB, K, K)];
        // the diagonal is element r of lanes c == 4g + r
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (c == 4 * g + r && (K < NB - 1 || c < nlast)) t[r] -= lam_n;
        *reinterpret_cast<f4*>(&S.T[c * 16 + 4 * g]) = t;
    }
    static __device__ __forceinline__ void panel(f4 (&acc)[ntiles(NB)], SolveLds<NB>& S,
                                                 int nlast, int lane) {
        if constexpr (K < NB - 1) {
            const int g = lane >> 4, c = lane & 15;
            f4 wop;   // element s: -W_K[c][4g + s] (the tiles hold -U)
#pragma unroll
            for (int s = 0; s < 4; ++s) wop[s] = S.W[K][(4 * g + s) * 16 + c];
#pragma unroll
            for (int I = K + 1; I < NB; ++I) {
                f4 d = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    d = __builtin_amdgcn_mfma_f32_16x16x4f32(wop[s], acc[tu(NB, K, I)][s], d,
                                                             0, 0, 0);
                acc[tu(NB, K, I)] = d;
            }
            if (c == nlast)   // y_K: the augmented column of the last panel tile
                *reinterpret_cast<f4*>(&S.y[16 * K + 4 * g]) = acc[tu(NB, K, NB - 1)];
#pragma unroll
            for (int J = K + 1; J < NB; ++J)
#pragma unroll
                for (int I = J; I < NB; ++I)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        acc[tu(NB, J, I)] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            acc[tu(NB, K, J)][s], acc[tu(NB, K, I)][s], acc[tu(NB, J, I)], 0,
                            0, 0);
        }
    }
    static __device__ __forceinline__ f4 matvec(const f4 (&acc)[ntiles(NB)],
                                                const SolveLds<NB>& S, int lane) {
        const int c = lane & 15;
        f4 part = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int I = K + 1; I < NB; ++I) part += acc[tu(NB, K, I)] * S.x[16 * I + c];
        return part;
    }
};

// run-time K -> Block<NB, K>.  Each case ends in its own empty asm statement so that the
// optimiser cannot merge the cases into one access with a run-time tile index (which would move
// the accumulator tiles out of registers).
template <int K>
__device__ __forceinline__ void case_marker() {
    asm volatile("; als block case %0" ::"n"(K));
}
template <int NB, int K = 0>
__device__ __forceinline__ void stage_diag(int k, const f4 (&acc)[ntiles(NB)], SolveLds<NB>& S,
                                           float lam_n, int nlast, int lane) {
    if (k == K) {
        Block<NB, K>::stage(acc, S, lam_n, nlast, lane);
        case_marker<K>();
    } else if constexpr (K + 1 < NB) {
        stage_diag<NB, K + 1>(k, acc, S, lam_n, nlast, lane);
    }
}
template <int NB, int K = 0>
__device__ __forceinline__ void panel_update(int k, f4 (&acc)[ntiles(NB)], SolveLds<NB>& S,
                                             int nlast, int lane) {
    if (k == K) {
        Block<NB, K>::panel(acc, S, nlast, lane);
        case_marker<K>();
    } else if constexpr (K + 1 < NB - 1) {
        panel_update<NB, K + 1>(k, acc, S, nlast, lane);
    }
}
template <int NB, int K = 0>
__device__ __forceinline__ f4 back_matvec(int k, const f4 (&acc)[ntiles(NB)],
                                          const SolveLds<NB>& S, int lane) {
    if (k == K) {
        const f4 r = Block<NB, K>::matvec(acc, S, lane);
        case_marker<K>();
        return r;
    }
    if constexpr (K + 1 < NB) return back_matvec<NB, K + 1>(k, acc, S, lane);
    return f4{0.f, 0.f, 0.f, 0.f};
}

// Regularise and solve, in place on the accumulator tiles (upper block-triangle of the
// augmented matrix M = [A b; b^T .]).  Blocked right-looking Cholesky over the 16-column blocks:
// factor and invert the diagonal tile (factor_tile), then panel and trailing update by MFMA
// (Block::panel).  The augmented column carries b through the same updates, so its entries
// become y = L^{-1} b.  Back substitution x_K = W_K^T (y_K - sum_{I>K} D_{K,I} x_I) runs last
// block first.  Only real pivots (rows < f) are factored; the last block's padding is the
// identity.  Returns false if a pivot was not positive; leaves the solution in S.x (zero past
// f).
template <int NB>
__device__ __forceinline__ bool solve_core(f4 (&acc)[ntiles(NB)], int f, float lam_n,
                                           SolveLds<NB>& S, int lane) {
    const int g = lane >> 4, c = lane & 15;
    const int nlast = f - 16 * (NB - 1);   // real columns of the last block; b is its column nlast
    // -M: the factorisation below keeps unfactored tiles negated (the regularisation joins each
    // diagonal tile as it is staged)
#pragma unroll
    for (int t = 0; t < ntiles(NB); ++t) acc[t] = -acc[t];

    int pmin = 0x7FFFFFFF, pmax = 0;
    // unrolled: with a run-time block loop every block's results had to be copied back into the
    // loop-carried registers (about 110 register-pair moves per row)
#pragma unroll
    for (int K = 0; K < NB; ++K) {
        stage_diag<NB>(K, acc, S, lam_n, nlast, lane);
        __syncthreads();
        if (K == NB - 1 && nlast <= 4)
            factor_tile<NB, false>(S, K, nlast, nlast, pmin, pmax, lane);
        else
            factor_tile<NB, true>(S, K, (K < NB - 1) ? 16 : nlast, nlast, pmin, pmax, lane);
        __syncthreads();
        panel_update<NB>(K, acc, S, nlast, lane);
    }
    const bool ok = pmin > 0 && pmax < 0x7F800000;   // every pivot positive and finite
    // back substitution, last block first; x is zero past f (b column and padding).  Lane
    // (g, c < 4) finishes entry kk = 4g + c of the block (the transposed row sums put it there);
    // with -W_K in S.W, it works with -z.
    for (int j = lane; j < 16 * NB; j += kWave) S.x[j] = 0.f;
    __syncthreads();
    const int kq = 4 * g + (c & 3);
#pragma unroll
    for (int K = NB - 1; K >= 0; --K) {
        const bool real = K < NB - 1 || kq < nlast;
        const float part = row_sum16_t(back_matvec<NB>(K, acc, S, lane));
        const float nz = real ? part - S.y[16 * K + kq] : 0.f;   // -z[kq]
        if (c < 4) S.z[kq] = nz;
        __syncthreads();
        const float zc = S.z[c];
        f4 xs;
#pragma unroll
        for (int s = 0; s < 4; ++s) xs[s] = S.W[K][(4 * g + s) * 16 + c] * zc;
        const float xv = row_sum16_t(xs);
        if (c < 4) S.x[16 * K + kq] = real ? xv : 0.f;
        __syncthreads();
    }
    return ok;
}

// ---- rows with a column of tiny values
//
// bf16 has fp32's exponents but no smaller subnormals than 2^-133, so a value below about 2^-110 loses
// low bits with its parts.  That shows where all of a row's ratings, or a whole column of its gathered
// factors, are that small (beside larger ones the loss is below 2^-24 of the column).  Then x_u, or
// its entry for the column, is tiny too: at most the column's norm times that of the ratings over
// lambda n_u (the ridge residual is no larger than the ratings), which is below kTinyX unless the
// ratings exceed lambda 2^60-fold.  Rows with such an entry are set aside by k_herm_solve and summed
// again with fp32 products, whose range is fp32's, in k_reduce_solve.  (With lambda = 0 such a column's
// pivot underflows, and x_u is NaN either way.)  Rows with a zero in x_u are set aside as well.
constexpr float kTinyX = 0x1p-40f;
constexpr unsigned kSetAside = 0x7FA5A5A5u;   // a NaN that no solve writes: first value of a row set aside

// The augmented Gram matrix of a row's entries [beg, end) with fp32 products, four entries a step;
// the accumulators are rounded once per 16 entries.
template <int NB>
__device__ __forceinline__ void plain_row(f4 (&acc)[ntiles(NB)], const int32_t* __restrict__ colidx,
                                          const float* __restrict__ vals,
                                          const float* __restrict__ theta, int f, int64_t beg,
                                          int64_t end, int lane) {
    constexpr int kSteps = 4;
    const int g = lane >> 4, c = lane & 15;
#pragma unroll
    for (int t = 0; t < ntiles(NB); ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    for (int64_t k = beg; k < end; k += 4 * kSteps) {
        float x[kSteps][NB];
#pragma unroll
        for (int j = 0; j < kSteps; ++j) {
            const int64_t e = k + 4 * j + g;
            const bool valid = e < end;
            const float* row = theta + (valid ? (size_t)(unsigned)colidx[e] * (size_t)f : 0);
            const float r = valid ? vals[e] : 0.f;
#pragma unroll
            for (int I = 0; I < NB; ++I) {
                const int v = 16 * I + c;
                x[j][I] = valid && v < f ? row[v] : (v == f ? r : 0.f);
            }
        }
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
            for (int J = I; J < NB; ++J) {
                f4 t = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < kSteps; ++j)
                    t = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j][I], x[j][J], t, 0, 0, 0);
                acc[tu(NB, I, J)] += t;
            }
    }
}

// solve_core, then x_u (f floats, NaN if a pivot was not positive) to xrow.  tiny: whether an entry of
// x_u is below kTinyX.
template <int NB>
__device__ __forceinline__ bool solve_row(f4 (&acc)[ntiles(NB)], int f, float lam_n,
                                          SolveLds<NB>& S, float* __restrict__ xrow, int lane,
                                          bool& tiny) {
    const bool ok = solve_core<NB>(acc, f, lam_n, S, lane);
    bool below = false;
    for (int j = lane; j < f; j += kWave) {
        const float x = ok ? S.x[j] : __builtin_nanf("");
        below |= __builtin_fabsf(x) < kTinyX;
        xrow[j] = x;
    }
    tiny = __ballot(below) != 0;
    return ok;
}

template <int NB>
__device__ __forceinline__ void write_zero_row(float* __restrict__ xrow, int f, int lane) {
    for (int j = lane; j < f; j += kWave) xrow[j] = 0.f;
}

// ------------------------------------------------------------------------ kernels --------

// Persistent waves claim chunks in order (see kStripes); chunk c covers the entries from
// bounds[c] to bounds[c+1].  Whole rows are solved here; the piece of a row cut at the start of
// the chunk goes to slot 2c, the piece cut at its end to slot 2c+1, so what is stored where does
// not depend on which wave ran the chunk.  Rows are software-pipelined: the next piece's index
// batches load while this piece's Gram runs, and its first theta gathers are in flight while
// this piece is solved.
struct Piece {
    int64_t u, beg, end;   // row, entry range [beg, end)
    bool whole;            // the chunk holds the whole row
};

// Bit j set: chunk first + j (j < kSmallPerWave) is not empty.
__device__ __forceinline__ unsigned nonempty_chunks(const int64_t* __restrict__ bounds, int first,
                                                    int lane) {
    const int j = lane < kSmallPerWave ? lane : kSmallPerWave - 1;
    const int64_t* b = bounds + 2 * (int64_t)(first + j);
    const bool some = b[0] != b[2] || b[1] != b[3];
    return (unsigned)__ballot(some && lane < kSmallPerWave);
}

// The next chunk of a stripe, from its counter; C or more when it is used up.  Every lane takes part
// in the claim (lane 0 adds one, the others zero).
__device__ __forceinline__ int claim_chunk(unsigned* __restrict__ ctr, int stripes, int stripe,
                                           int lane) {
    const unsigned got = atomicAdd(ctr + stripe * kStripeWords, lane == 0 ? 1u : 0u);
    return __builtin_amdgcn_readfirstlane((int)got) * stripes + stripe;
}

template <int NB, int BUF, int LAST, bool PARTS>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(gram_waves(NB, LAST))))
void k_herm_solve(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ vals, const float* __restrict__ theta, int64_t m, int64_t n,
    int f, float lambda, int C, const int64_t* __restrict__ bounds, float* __restrict__ x_out,
    float* __restrict__ slots, float* __restrict__ wave_slots, int part_mask, int64_t c_row,
    unsigned long long* __restrict__ nonspd, unsigned* __restrict__ chunk_ctr,
    unsigned* __restrict__ set_aside) {
    // Where a piece may be longer than a part, both instantiations (with and without parts) are
    // launched, and the one that does not match this call returns at once.  A piece lies within a chunk and within a row: a chunk holds at
    // most ceil(T1 / W) cost units (c_nnz per entry) plus the snapping of its two cut offsets,
    // and a row at most n entries (its columns are distinct).
    {
        const int64_t T = kCostPerEntry * rowptr[m] + c_row * m;
        int64_t longest = (T / (int64_t)gridDim.x + 1) / kCostPerEntry + 2 * kSnap + 1;
        if (longest > n) longest = n;
        if ((longest > (int64_t)kGroupEntries * (part_mask + 1)) != PARTS) return;
    }
    using G = Gather<NB, BUF, LAST>;
    __shared__ __attribute__((aligned(16))) SolveLds<NB> lds;
    __shared__ typename G::Entry ring[kGramRing];
    __shared__ __attribute__((aligned(16))) float stage[BUF == kFormStaged ? stage_floats(NB) : 4];
    const int lane = threadIdx.x;
    if constexpr (BUF == kFormStaged) {
        for (int i = lane; i < stage_floats(NB); i += kWave) stage[i] = 0.f;
        __syncthreads();
    }
    const G gat(theta, n, f, lane & 15, stage);
    const int q = f - 16 * (NB - 1) + 1, third = (lane & 15) / q;
    static_assert(NB * kWave * sizeof(f4) <= sizeof(SolveLds<NB>),
                  "fold_packed and fold_rating reuse the solve's LDS");
    float* __restrict__ wslot = wave_slots + (size_t)blockIdx.x * slot_floats(NB);
    // No lane-0-only region in the claim loop: every lane takes part in a claim, and the wave's
    // count of non-SPD rows stays in a register until the
    // loop has ended (a lane-0 region at each end of a loop body can be joined across the back
    // edge, leaving lanes 1..63 in a loop of their own).
    unsigned bad = 0;
    const int W = (int)gridDim.x, self = (int)blockIdx.x;
    const bool fixed = kCostPerEntry * rowptr[m] + c_row * m <=
                       static_entries(NB) * kCostPerEntry * (int64_t)W;
    bool first = true;
    const int stripes = W >= 8 * kStripes ? kStripes : 1;   // each with waves of its own
    const int stripe = (self >> 3) & (stripes - 1);
    unsigned small = 0;                                     // the wave's small chunks to run
    for (;;) {
        int c;
        if (fixed) {
            if (first) {
                c = self;
                if (C > W) small = nonempty_chunks(bounds, W + kSmallPerWave * self, lane);
            } else {
                if (small == 0) break;
                c = W + kSmallPerWave * self + __builtin_ctz(small);
                small &= small - 1;
            }
            first = false;
        } else {
            c = claim_chunk(chunk_ctr, stripes, stripe, lane);
            if (c >= C) break;
        }
        const int64_t u0 = bounds[2 * c], k0 = bounds[2 * c + 1];
        const int64_t u1 = bounds[2 * c + 2], k1 = bounds[2 * c + 3];
        // the first piece with entries at or after row u; empty rows on the way get x_u = 0
        auto next_piece = [&](int64_t u, Piece& p) -> bool {
            for (; u <= u1 && u < m; ++u) {
                const int64_t rs = rowptr[u], nu = rowptr[u + 1] - rs;
                const int64_t ka = (u == u0) ? k0 : 0;
                int64_t kb = nu;
                if (u == u1) {
                    if (k1 == 0) return false;
                    kb = k1;
                }
                if (nu == 0) {
                    write_zero_row<NB>(x_out + (size_t)u * f, f, lane);
                    continue;
                }
                if (ka >= kb) continue;
                p = Piece{u, rs + ka, rs + kb, ka == 0 && kb == nu};
                return true;
            }
            return false;
        };
        Piece cur;
        if (!next_piece(u0, cur)) continue;
        typename G::Entry first_batch =
            load_entry<kGramBatch>(gat, colidx, vals, cur.beg, cur.end - cur.beg, 0, lane);
        Raw<G> raw;
        int slot = 0;
        start_piece(gat, first_batch, ring, slot, lane, raw);
        for (;;) {
            Piece nxt;
            const bool more = next_piece(cur.u + 1, nxt);
            if (more)
                first_batch =
                    load_entry<kGramBatch>(gat, colidx, vals, nxt.beg, nxt.end - nxt.beg, 0, lane);
            f4 acc[ntiles(NB)];
            GramBody<NB, LAST, G, PARTS> body{part_mask, gat, acc, q, third, &lds, wslot, lane};
            body.clear();
            group_loop(gat, colidx, vals, cur.beg, cur.end, ring, slot, lane, raw, more,
                       first_batch, body);
            body.finish();
            // a piece longer than a part: its earlier parts' sum is in the wave's slot
            if constexpr (PARTS) {
                if (cur.end - cur.beg > (int64_t)kGroupEntries * (part_mask + 1))
                    add_slot_in_fours<NB>(acc, wslot, lane);
            }
            // the solve is a latency-bound chain; raised priority lets it win issue slots over
            // the other wave's independent Gram MFMAs, which then fill the solve's gaps
            __builtin_amdgcn_s_setprio(2);
            if (cur.whole) {
                const int64_t nu = cur.end - cur.beg;
                const float lam_n = (float)((double)lambda * (double)nu);
                bool tiny;
                // (its LDS addresses are made per row in the parts form, which has no registers to keep
                // them in; spilled, they were 51 loads a row: music item side 27.5 -> 32 ms)
                if (!solve_row<NB>(acc, f, lam_n, lds, x_out + (size_t)cur.u * f,
                                   PARTS ? fresh_lane() : lane, tiny))
                    ++bad;
                if (__builtin_expect(tiny, 0)) {   // (every lane stores the same value)
                    x_out[(size_t)cur.u * f] = __builtin_bit_cast(float, kSetAside);
                    *set_aside = 1u;
                }
            } else {
                const int which = (cur.u == u0) ? 0 : 1;
                store_slot<NB>(acc, slots + (size_t)(2 * c + which) * slot_floats(NB), lane);
            }
            __builtin_amdgcn_s_setprio(0);
            if (!more) break;
            cur = nxt;
        }
    }
    bad = __builtin_amdgcn_readfirstlane(bad);
    if (bad) atomicAdd(nonspd, lane == 0 ? (unsigned long long)bad : 0ull);
}

// Rows cut by chunk boundaries.  Row u's pieces are: the first, held by chunk b_first - 1 (as
// that chunk's first piece if it started in row u, else as its last), then the piece starting at
// each boundary b_first..b_last that cuts u, in slot 2b (empty, and unwritten, when several
// boundaries snapped to one cut point).  The boundaries cutting one row are consecutive, so both
// ends are found by search over the sorted bounds.  A long row with more than kPieceGroup
// boundaries (sums_in_groups) is summed in two passes: every kPieceGroup-th boundary leads a group and sums
// the group's pieces, in chunk order, into its own slot; then the row's first boundary adds the
// first piece and the group sums, in order, and solves.  The order is fixed, so the result does
// not depend on timing.
constexpr int kPieceGroup = 16;
// Rows summed in two passes: those of more than kPieceGroup boundaries and long enough for as many
// pieces (cut points lie kSnap entries apart; a short sweep's chunks are smaller than that, and
// hundreds of boundaries fall on a few cut points).  An iteration on 1M ratings at f = 40, both
// reduce kernels of both sides: 78 us when every row of more than 16 boundaries took two passes and
// boundaries were looked at one by one, 54 us now.
__device__ __forceinline__ bool sums_in_groups(int boundaries, int64_t nu) {
    return boundaries > kPieceGroup && nu > (int64_t)kPieceGroup * kSnap;
}
// Blocks of the reduce kernels.  One per boundary cost 9 us a kernel where no row is cut (tiny,
// C = 36,864); 2,048 (all resident at f = 100) leave each wave up to nine cut rows one after the
// other: 133 us against 95 for k_reduce_solve on the movie user side, and 296 us against 264 for a
// whole iteration on 1M ratings at f = 40.  With 8,192 the tiny call takes 23.3 us, with 2,048 21.2.
constexpr int kReduceWaves = 8192;

__device__ __forceinline__ bool cuts_row(const int64_t* __restrict__ rowptr, int64_t m,
                                         const int64_t* __restrict__ bounds, int b) {
    const int64_t u = bounds[2 * b], k = bounds[2 * b + 1];
    return u < m && k > 0 && k < rowptr[u + 1] - rowptr[u];
}

// First and last boundary in [1, C-1] that cut row u, given that boundary b does.  Boundaries
// with row u and an offset strictly inside it form one run around b (bounds are sorted by (row,
// offset): one of row u at offset 0 precedes the run, one at n_u follows it).  Most runs hold one
// or two boundaries, so each end is found by galloping out from b (steps 1, 2, 4, ...) and then
// bisecting the last step: a few dependent loads for a short run instead of a bisection of all C.
__device__ __forceinline__ void cut_range(const int64_t* __restrict__ rowptr, int64_t m,
                                          const int64_t* __restrict__ bounds, int C, int b,
                                          int64_t u, int& b_first, int& b_last) {
    const auto in_run = [&](int x) { return bounds[2 * x] == u && cuts_row(rowptr, m, bounds, x); };
    int in = b, out = 0;   // in the run / below it (0: no boundary below the range)
    for (int d = 1;; d <<= 1) {
        const int x = b - d;
        if (x < 1) break;
        if (!in_run(x)) {
            out = x;
            break;
        }
        in = x;
    }
    while (in - out > 1) {
        const int mid = (in + out) >> 1;
        if (in_run(mid)) in = mid; else out = mid;
    }
    b_first = in;
    in = b;
    out = C;               // above the run (C: no boundary above the range)
    for (int d = 1;; d <<= 1) {
        const int x = b + d;
        if (x > C - 1) break;
        if (!in_run(x)) {
            out = x;
            break;
        }
        in = x;
    }
    while (out - in > 1) {
        const int mid = (in + out) >> 1;
        if (in_run(mid)) in = mid; else out = mid;
    }
    b_last = in;
}

// Add the non-empty boundary pieces of row u for boundaries bb in [from, to] into acc, in order (the
// piece of chunk bb runs to the next boundary in the row, or to the row's end).  A wave looks at 64
// boundaries at once: in a short sweep most of a row's boundaries fall on the same few cut points.
template <int NB>
__device__ __forceinline__ void add_pieces(f4 (&acc)[ntiles(NB)], const int64_t* __restrict__ bounds,
                                           const float* __restrict__ slots, int from, int to,
                                           int b_last, int64_t nu, int lane) {
    for (int base = from; base <= to; base += kWave) {
        const int x = base + lane;
        const bool some =
            x <= to && bounds[2 * x + 1] < (x < b_last ? bounds[2 * (x + 1) + 1] : nu);
        uint64_t todo = __ballot(some);
        while (todo) {
            const int bb = base + __builtin_ctzll(todo);
            todo &= todo - 1;
            add_slot<NB>(acc, slots + (size_t)(2 * bb) * slot_floats(NB), lane);
        }
    }
}

// The internal boundaries 1 .. C - 1 are dealt to the waves of the grid in turn (wave j: 1 + j,
// 1 + j + grid, ...).  A wave looks at 64 of its boundaries at once, a lane each, and takes up those
// that cut a row one after the other.
template <class Pick, class Take>
__device__ __forceinline__ void for_boundaries(int C, int lane, Pick&& pick, Take&& take) {
    const int grid = (int)gridDim.x;
    for (int64_t b0 = 1 + (int64_t)blockIdx.x; b0 < C; b0 += (int64_t)grid * kWave) {
        const int64_t b = b0 + (int64_t)lane * grid;
        uint64_t todo = __ballot(b < C && pick((int)b));
        while (todo) {
            const int l = __builtin_ctzll(todo);
            todo &= todo - 1;
            take((int)(b0 + (int64_t)l * grid));
        }
    }
}

// Pass 1: group leaders of long cut rows sum their group.  A boundary's row has more than
// kPieceGroup boundaries only if some kPieceGroup - 1 away or nearer lies in it too.
template <int NB>
__global__ __launch_bounds__(kWave) void k_reduce_groups(
    const int64_t* __restrict__ rowptr, int64_t m, int C, const int64_t* __restrict__ bounds,
    float* __restrict__ slots) {
    const int lane = threadIdx.x;
    const auto pick = [&](int b) {
        if (!cuts_row(rowptr, m, bounds, b)) return false;
        const int64_t u = bounds[2 * b];
        if (!sums_in_groups(kPieceGroup + 1, rowptr[u + 1] - rowptr[u])) return false;
        return (b > 1 && bounds[2 * (b - 1)] == u) || (b + 1 < C && bounds[2 * (b + 1)] == u);
    };
    for_boundaries(C, lane, pick, [&](int b) {
        const int64_t u = bounds[2 * b];
        int b_first, b_last;
        cut_range(rowptr, m, bounds, C, b, u, b_first, b_last);
        if (!sums_in_groups(b_last - b_first + 1, rowptr[u + 1] - rowptr[u]) ||
            (b - b_first) % kPieceGroup != 0)
            return;
        f4 acc[ntiles(NB)];
#pragma unroll
        for (int t = 0; t < ntiles(NB); ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
        const int to = b + kPieceGroup - 1 < b_last ? b + kPieceGroup - 1 : b_last;
        add_pieces<NB>(acc, bounds, slots, b, to, b_last, rowptr[u + 1] - rowptr[u], lane);
        store_slot<NB>(acc, slots + (size_t)(2 * b) * slot_floats(NB), lane);
    });
}

// Pass 2: the first boundary that cuts a row sums its pieces (or its group sums) and solves it.
template <int NB>
__device__ __forceinline__ void reduce_row(const int64_t* __restrict__ rowptr,
                                           const int32_t* __restrict__ colidx,
                                           const float* __restrict__ vals,
                                           const float* __restrict__ theta, int64_t m, int C, int f,
                                           float lambda, const int64_t* __restrict__ bounds,
                                           float* __restrict__ x_out,
                                           const float* __restrict__ slots, unsigned& bad,
                                           SolveLds<NB>& lds, int b, int lane) {
    const int64_t u = bounds[2 * b], nu = rowptr[u + 1] - rowptr[u];
    // the row's last boundary: most rows have few, looked at side by side
    const int x = b + 1 + lane;
    const uint64_t run =
        __ballot(x < C && bounds[2 * x] == u && bounds[2 * x + 1] > 0 && bounds[2 * x + 1] < nu);
    int b_first = b, b_last = b + __builtin_ctzll(~run);
    if (run == ~0ull) cut_range(rowptr, m, bounds, C, b, u, b_first, b_last);
    f4 acc[ntiles(NB)];
#pragma unroll
    for (int t = 0; t < ntiles(NB); ++t) acc[t] = f4{0.f, 0.f, 0.f, 0.f};
    // chunk b-1 holds the row's first piece: as its first piece if it started in row u
    // (then at entry 0), else as its last piece
    const int first_slot = (bounds[2 * (b - 1)] == u) ? 2 * (b - 1) : 2 * (b - 1) + 1;
    add_slot<NB>(acc, slots + (size_t)first_slot * slot_floats(NB), lane);
    if (!sums_in_groups(b_last - b_first + 1, nu)) {
        add_pieces<NB>(acc, bounds, slots, b, b_last, b_last, nu, lane);
    } else {
        for (int g = b; g <= b_last; g += kPieceGroup)
            add_slot<NB>(acc, slots + (size_t)(2 * g) * slot_floats(NB), lane);
    }
    const float lam_n = (float)((double)lambda * (double)nu);
    for (bool tiny = false, again = false;; again = true) {
        if (again) plain_row<NB>(acc, colidx, vals, theta, f, rowptr[u], rowptr[u + 1], lane);
        if (!solve_row<NB>(acc, f, lam_n, lds, x_out + (size_t)u * f, lane, tiny)) ++bad;
        if (again || !tiny) break;
    }
}

// The rows that k_herm_solve has set aside: a wave looks at 64 rows at once.
template <int NB>
__device__ __forceinline__ void solve_set_aside(const int64_t* __restrict__ rowptr,
                                                const int32_t* __restrict__ colidx,
                                                const float* __restrict__ vals,
                                                const float* __restrict__ theta, int64_t m, int f,
                                                float lambda, float* __restrict__ x_out,
                                                unsigned& bad, SolveLds<NB>& lds, int lane) {
    for (int64_t u0 = (int64_t)blockIdx.x * kWave; u0 < m; u0 += (int64_t)gridDim.x * kWave) {
        const int64_t u = u0 + lane;
        uint64_t todo = __ballot(
            u < m && reinterpret_cast<const unsigned*>(x_out)[(size_t)u * f] == kSetAside);
        while (todo) {
            const int64_t v = u0 + __builtin_ctzll(todo);
            todo &= todo - 1;
            const int64_t beg = rowptr[v], end = rowptr[v + 1];
            f4 acc[ntiles(NB)];
            plain_row<NB>(acc, colidx, vals, theta, f, beg, end, lane);
            const float lam_n = (float)((double)lambda * (double)(end - beg));
            bool tiny;
            if (!solve_row<NB>(acc, f, lam_n, lds, x_out + (size_t)v * f, lane, tiny)) ++bad;
        }
    }
}

template <int NB>
__global__ __launch_bounds__(kWave) void k_reduce_solve(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ vals, const float* __restrict__ theta, int64_t m, int C, int f,
    float lambda, const int64_t* __restrict__ bounds, float* __restrict__ x_out,
    const float* __restrict__ slots, unsigned long long* __restrict__ nonspd,
    const unsigned* __restrict__ set_aside) {
    __shared__ __attribute__((aligned(16))) SolveLds<NB> lds;
    const int lane = threadIdx.x;
    unsigned bad = 0;   // non-SPD rows of this wave, added once after the loop
    const auto first_cut = [&](int b) {
        if (!cuts_row(rowptr, m, bounds, b)) return false;
        return !(b > 1 && bounds[2 * (b - 1)] == bounds[2 * b] &&
                 cuts_row(rowptr, m, bounds, b - 1));
    };
    for_boundaries(C, lane, first_cut, [&](int b) {
        reduce_row<NB>(rowptr, colidx, vals, theta, m, C, f, lambda, bounds, x_out, slots, bad,
                       lds, b, lane);
    });
    if (*set_aside)
        solve_set_aside<NB>(rowptr, colidx, vals, theta, m, f, lambda, x_out, bad, lds, lane);
    bad = __builtin_amdgcn_readfirstlane(bad);
    if (bad) atomicAdd(nonspd, lane == 0 ? (unsigned long long)bad : 0ull);
}

// RMSE body: per step, entry slot g's residual r - x_u . theta_v in fp32 (the dot product over
// the slot's 16 lanes by DPP row sums); the squares of a group's kGroup steps are summed in fp32
// (at most kGroup terms per lane) and that sum is added in fp64 by the slot's first lane at the
// group's last step.  An entry past the piece's end gathers zeros and rating 0, so its residual
// is 0.  x_u sits in registers: lane (g, c) holds x_u[16 I + c] (0 past f, which also cancels the
// rating that the gather puts in column f).
template <int NB, class G>
struct RmseBody {
    const G& gat;
    const float (&xr)[NB];
    double& acc;
    bool lead;
    float v[NB], r;
    float sq;   // this group's squares so far
    __device__ __forceinline__ void take(const float (&B)[G::kBuf], float rr, bool ok) {
        gat.operands(B, rr, v);
        r = ok ? rr : 0.f;
    }
    template <int J>
    __device__ __forceinline__ void run() {
        float d = 0.f;
#pragma unroll
        for (int I = 0; I < NB; ++I) d = __builtin_fmaf(v[I], xr[I], d);
        d = row_sum16(d);
        const float e = r - d;
        sq = (J == 0) ? e * e : __builtin_fmaf(e, e, sq);
        if constexpr (J == kGroup - 1) acc += lead ? (double)sq : 0.0;
    }
};

// RMSE partials: the entries are cut into C equal chunks, chunk w = [nnz w / C, nnz (w+1) / C);
// a grid of one wave per chunk takes chunk w in block w; a narrower one claims chunks in order from
// a counter (about 11.5 ns per claim on its one address: the 8,192 + 8,192 claims of a full-width
// grid took 0.19 ms, all of the time of a call on 1M ratings).  Each chunk is walked row piece by
// row piece through the gather pipeline (the next piece's index batches load during the current piece;
// x_u is loaded once per piece).  Chunk w's fp64 sum goes to partial[w], so the result does not
// depend on how many waves run or which wave took which chunk: the kernel may run at any width,
// e.g. one wave per SIMD beside a half-sweep.  NB = f / 16 + 1 (the gather's block count).
template <int NB, bool BUF>
__global__ __launch_bounds__(kWave) void k_rmse_rows(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ vals, int64_t m, int64_t n, int f, const float* __restrict__ x,
    const float* __restrict__ theta, int C, double* __restrict__ partial,
    unsigned* __restrict__ claim) {
    using G = Gather<NB, BUF ? kFormBuffer : kFormGlobal>;
    __shared__ typename G::Entry ring[kRing];
    const int lane = threadIdx.x, c = lane & 15;
    const int64_t nnz = rowptr[m];
    // No lane-0-only region in this loop: every lane takes part in the claim (lane 0 adds one,
    // the others zero) and every lane stores the wave's sum.  (Two lane-0 regions at the ends of
    // the loop body were joined across the back edge by the compiler, leaving lanes 1..63 in a
    // loop of their own that read a stale chunk number.)
    const bool claims = (int)gridDim.x < C;
    for (int turn = 0;; ++turn) {
        int w;
        if (claims) {
            const unsigned got = atomicAdd(claim, lane == 0 ? 1u : 0u);
            w = __builtin_amdgcn_readfirstlane((int)got);
        } else {
            w = turn == 0 ? (int)blockIdx.x : C;
        }
        if (w >= C) break;
        const int64_t kb = nnz / C * w + (nnz % C) * w / C;
        const int64_t ke = nnz / C * (w + 1) + (nnz % C) * (w + 1) / C;
        double acc = 0.0;
        if (kb < ke) {
            int64_t lo = 0, hi = m - 1;   // row of entry kb: largest u < m with rowptr[u] <= kb
            while (lo < hi) {
                const int64_t mid = (lo + hi + 1) >> 1;
                if (rowptr[mid] <= kb) lo = mid; else hi = mid - 1;
            }
            int64_t u = lo;
            int64_t pb = kb, pe = rowptr[u + 1] < ke ? rowptr[u + 1] : ke;
            const G gat(theta, n, f, c);
            RowIndex<G> ix;
            Inflight<G::kBuf> in;
            gram_prefetch(gat, colidx, vals, pb, pe, lane, ix);
            gram_stage(gat, ix, ring, lane, in);
            for (;;) {
                int64_t un = u + 1;   // the next row with entries in the range
                while (un < m && rowptr[un] < ke && rowptr[un + 1] == rowptr[un]) ++un;
                const bool more = un < m && rowptr[un] < ke;
                int64_t nb0 = 0, nb1 = 0;
                if (more) {
                    nb0 = rowptr[un];
                    nb1 = rowptr[un + 1] < ke ? rowptr[un + 1] : ke;
                    gram_prefetch(gat, colidx, vals, nb0, nb1, lane, ix);
                }
                float xr[NB];
#pragma unroll
                for (int I = 0; I < NB; ++I) {
                    const int j = 16 * I + c;
                    xr[I] = j < f ? x[(size_t)u * (size_t)f + j] : 0.f;
                }
                RmseBody<NB, G> body{gat, xr, acc, c == 0, {}, 0.f, 0.f};
                pipe_loop(gat, colidx, vals, pb, pe, ring, lane, in, body);
                if (!more) break;
                gram_stage(gat, ix, ring, lane, in);
                u = un;
                pb = nb0;
                pe = nb1;
            }
        }
        // only the 16-lane groups' first lanes hold sums: the full butterfly leaves the wave's
        // total in every lane
        for (int o = 1; o < kWave; o <<= 1) acc += __shfl_xor(acc, o);
        partial[w] = acc;
    }
}

// The partials' sum in a fixed order: thread t adds partials t, t + 1024, ..., then a butterfly
// per wave and the waves in order.  (One wave with 128 loads, each waited for, took 33-42 us.)
constexpr int kFinalThreads = 1024;

__global__ __launch_bounds__(kFinalThreads) void k_rmse_final(const int64_t* __restrict__ rowptr,
                                                              int64_t m, int W,
                                                              const double* __restrict__ partial,
                                                              double* __restrict__ out) {
    __shared__ double sums[kFinalThreads / kWave];
    const int t = threadIdx.x;
    double s = 0.0;
#pragma unroll 8
    for (int i = t; i < W; i += kFinalThreads) s += partial[i];
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    if ((t & (kWave - 1)) == 0) sums[t / kWave] = s;
    __syncthreads();
    if (t == 0) {
        double all = 0.0;
        for (int i = 0; i < kFinalThreads / kWave; ++i) all += sums[i];
        const int64_t nnz = rowptr[m];
        out[0] = nnz > 0 ? sqrt(all / (double)nnz) : 0.0;
    }
}

__global__ void k_reset_counter(unsigned long long* p) { *p = 0ull; }

// ------------------------------------------------------------------ CSR -> CSC -----------

// The transpose R -> R^T that the update-Theta half-sweep reads (eq. 3 is the same method on
// the columns of R).  Stable: within a column the entries keep the order of their rows.
// The rows are cut into R row blocks of about nnz / R entries each (whole rows; block b holds
// rows [tr_row_begin(b), tr_row_begin(b+1))).  cnt[b][v] counts block b's entries in column v;
// a prefix over b turns it into the offset of block b's first entry within column v, and one
// wave per block then walks its rows in order, so every column receives its rows ascending.
// Entries whose column lies outside [0, n) are skipped by every pass (the contract leaves them
// undefined; skipping keeps every access in bounds).

// First row of row block b: the smallest u with rowptr[u] >= floor(b nnz / R) (binary search).
__device__ __forceinline__ int64_t tr_row_begin(const int64_t* __restrict__ rowptr, int64_t m,
                                                int R, int b) {
    const int64_t nnz = rowptr[m];
    // floor(nnz b / R) without overflow: nnz = q R + r, r b < R^2
    const int64_t target = (nnz / R) * b + ((nnz % R) * b) / R;
    int64_t lo = 0, hi = m;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rowptr[mid] < target) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// The counting passes run when the sort (k_rx_*, below) does not: when there are more entries than
// `over`, the most that it takes.
__global__ __launch_bounds__(256) void k_tr_zero(const int64_t* __restrict__ rowptr, int64_t m,
                                                 int64_t over, int32_t* __restrict__ p,
                                                 int64_t count) {
    if (rowptr[m] <= over) return;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * 256)
        p[i] = 0;
}

// cnt[b][v] += 1 for every entry of row block b (one workgroup per block; the order of the
// increments does not matter).
__global__ __launch_bounds__(256) void k_tr_count(const int64_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ colidx, int64_t m,
                                                  int64_t n, int64_t over, int R,
                                                  int32_t* __restrict__ cnt) {
    if (rowptr[m] <= over) return;
    const int b = blockIdx.x;
    const int64_t k0 = rowptr[tr_row_begin(rowptr, m, R, b)];
    const int64_t k1 = rowptr[tr_row_begin(rowptr, m, R, b + 1)];
    int32_t* row = cnt + (size_t)b * (size_t)n;
    for (int64_t k = k0 + threadIdx.x; k < k1; k += 256) {
        const int32_t v = colidx[k];
        if (v >= 0 && v < n) atomicAdd(&row[v], 1);
    }
}

// Per column v (one thread each): cnt[b][v] <- the sum over b' < b, and colptr[v] <- the
// column's total (scanned over v afterwards).
__global__ __launch_bounds__(256) void k_tr_colscan(const int64_t* __restrict__ rowptr, int64_t m,
                                                    int64_t n, int64_t over, int R,
                                                    int32_t* __restrict__ cnt,
                                                    int64_t* __restrict__ colptr) {
    if (rowptr[m] <= over) return;
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= n) return;
    int32_t run = 0;
    for (int b = 0; b < R; ++b) {
        int32_t* c = cnt + (size_t)b * (size_t)n + v;
        const int32_t t = *c;
        *c = run;
        run += t;
    }
    colptr[v] = run;
}

// Exclusive scan of a[0, len) in place, a[len] <- the total: tile sums (kScanTile elements per
// workgroup), a scan of the tile sums by one workgroup, then each tile scanned with its offset.
constexpr int kScanPer = 16;
constexpr int kScanTile = 256 * kScanPer;

// Exclusive scan of one value per thread over a workgroup of 256 (4 waves); returns the prefix
// and sets *total.
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t x, int64_t* sh, int64_t* total) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int64_t inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int64_t base = 0;
    for (int i = 0; i < w; ++i) base += sh[i];
    *total = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return base + inc - x;
}

__global__ __launch_bounds__(256) void k_scan_sums(const int64_t* __restrict__ a, int64_t len,
                                                   int64_t* __restrict__ sums) {
    __shared__ int64_t sh[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t x = 0;
    for (int j = 0; j < kScanPer; ++j) {
        const int64_t i = base + (int64_t)threadIdx.x * kScanPer + j;
        if (i < len) x += a[i];
    }
    int64_t total;
    (void)block_exclusive_scan(x, sh, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_scan_top(int64_t* __restrict__ sums, int64_t tiles,
                                                  int64_t* __restrict__ a, int64_t len) {
    __shared__ int64_t sh[4];
    int64_t carry = 0;
    for (int64_t c = 0; c < tiles; c += 256) {
        const int64_t i = c + threadIdx.x;
        const int64_t x = i < tiles ? sums[i] : 0;
        int64_t total;
        const int64_t ex = block_exclusive_scan(x, sh, &total);
        if (i < tiles) sums[i] = carry + ex;
        carry += total;
    }
    if (threadIdx.x == 0) a[len] = carry;
}

__global__ __launch_bounds__(256) void k_scan_apply(int64_t* __restrict__ a, int64_t len,
                                                    const int64_t* __restrict__ sums) {
    __shared__ int64_t sh[4];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
    int64_t v[kScanPer];
    int64_t x = 0;
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        v[j] = base + j < len ? a[base + j] : 0;
        x += v[j];
    }
    int64_t total;
    int64_t run = sums[blockIdx.x] + block_exclusive_scan(x, sh, &total);
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) {
        if (base + j < len) a[base + j] = run;
        run += v[j];
    }
}

// LDS atomics whose result is not used may still be on their way at a barrier (the compiler leaves
// their wait out where they end a loop body, and counts of other waves were lost that way): waits
// for this wave's before it meets the others.
__device__ __forceinline__ void lds_atomics_done() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// LDS forms of the count and the scatter, for n <= kTrLdsCols: the block's per-column counters
// (cursors) live in the workgroup's LDS.  Counting: one workgroup of 256 per row block adds its
// entries into LDS and writes the n counts out.  Scatter: one wave per row block loads
// colptr[v] + cnt[b][v] into LDS and walks its rows in order; a wave's LDS atomics are performed
// in issue order, so a column's entries again arrive in row order.
constexpr int kTrLdsCols = 40960;   // 160 KB of int32 counters

__global__ __launch_bounds__(256) void k_tr_count_lds(const int64_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ colidx,
                                                      int64_t m, int n, int64_t over, int R,
                                                      int32_t* __restrict__ cnt) {
    if (rowptr[m] <= over) return;
    extern __shared__ int32_t lcnt[];
    const int b = blockIdx.x;
    for (int v = threadIdx.x; v < n; v += 256) lcnt[v] = 0;
    __syncthreads();
    const int64_t k0 = rowptr[tr_row_begin(rowptr, m, R, b)];
    const int64_t k1 = rowptr[tr_row_begin(rowptr, m, R, b + 1)];
    for (int64_t k = k0 + threadIdx.x; k < k1; k += 256) {
        const int32_t v = colidx[k];
        if (v >= 0 && v < n) atomicAdd(&lcnt[v], 1);
    }
    lds_atomics_done();
    __syncthreads();
    int32_t* row = cnt + (size_t)b * (size_t)n;
    for (int v = threadIdx.x; v < n; v += 256) row[v] = lcnt[v];
}

__global__ __launch_bounds__(kWave) void k_tr_scatter_lds(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ vals, int64_t m, int n, int64_t over, int R,
    const int32_t* __restrict__ cnt, const int64_t* __restrict__ colptr,
    int32_t* __restrict__ rowidx, float* __restrict__ vals_t) {
    if (rowptr[m] <= over) return;
    // cur[v]: where this block's next entry of column v goes -- its absolute position when
    // nnz < 2^31 (then no colptr read per entry), else its position within column v's run
    extern __shared__ int32_t cur[];
    const int b = blockIdx.x, lane = threadIdx.x;
    const bool absolute = rowptr[m] <= (int64_t)INT32_MAX;
    const int32_t* row = cnt + (size_t)b * (size_t)n;
    for (int v = lane; v < n; v += kWave)
        cur[v] = absolute ? (int32_t)(colptr[v] + row[v]) : row[v];
    __syncthreads();
    const int64_t u0 = tr_row_begin(rowptr, m, R, b), u1 = tr_row_begin(rowptr, m, R, b + 1);
    // chunks of up to 64 entries of one row, in order; the next chunk's column indices and
    // ratings load while this one is placed (a chunk never spans two rows, so the lanes of one
    // LDS atomic never share a column)
    int64_t u = u0, ks = 0, ke = 0;
    auto next_chunk = [&](int64_t& cu, int64_t& cs, int64_t& ce) {
        if (cs + kWave < ce) {
            cs += kWave;
            return;
        }
        for (++cu; cu < u1; ++cu) {
            cs = rowptr[cu];
            ce = rowptr[cu + 1];
            if (cs < ce) return;
        }
    };
    u = u0 - 1;
    next_chunk(u, ks, ke);   // the first chunk (ks + kWave >= ke = 0 starts the row walk)
    int32_t v = -1;
    float r = 0.f;
    if (u < u1 && ks + lane < ke) {
        v = colidx[ks + lane];
        r = vals[ks + lane];
    }
    while (u < u1) {
        int64_t nu = u, ns = ks, ne = ke;
        next_chunk(nu, ns, ne);
        int32_t nv = -1;
        float nr = 0.f;
        if (nu < u1 && ns + lane < ne) {
            nv = colidx[ns + lane];
            nr = vals[ns + lane];
        }
        if (ks + lane < ke && v >= 0 && v < n) {
            const int32_t at = atomicAdd(&cur[v], 1);
            const int64_t pos = absolute ? (int64_t)at : colptr[v] + at;
            rowidx[pos] = (int32_t)u;
            vals_t[pos] = r;
        }
        u = nu;
        ks = ns;
        ke = ne;
        v = nv;
        r = nr;
    }
}

// One wave per row block, its rows in order: each entry goes to colptr[v] + cnt[b][v], which
// then moves on by one.  The columns of one row are distinct, so the lanes of a row never share
// a counter; the fence after each row orders its counter updates before the next row's.
__global__ __launch_bounds__(kWave) void k_tr_scatter(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
    const float* __restrict__ vals, int64_t m, int64_t n, int64_t over, int R,
    int32_t* __restrict__ cnt, const int64_t* __restrict__ colptr, int32_t* __restrict__ rowidx,
    float* __restrict__ vals_t) {
    if (rowptr[m] <= over) return;
    const int b = blockIdx.x, lane = threadIdx.x;
    const int64_t u0 = tr_row_begin(rowptr, m, R, b), u1 = tr_row_begin(rowptr, m, R, b + 1);
    int32_t* row = cnt + (size_t)b * (size_t)n;
    for (int64_t u = u0; u < u1; ++u) {
        const int64_t k1 = rowptr[u + 1];
        for (int64_t k = rowptr[u] + lane; k < k1; k += kWave) {
            const int32_t v = colidx[k];
            if (v >= 0 && v < n) {
                const int32_t at = atomicAdd(&row[v], 1);
                const int64_t pos = colptr[v] + at;
                rowidx[pos] = (int32_t)u;
                vals_t[pos] = vals[k];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    }
}

// ---- the transpose as a stable radix sort by column (nnz up to what the workspace holds)
//
// What bounds the passes above is their scattered 4-byte stores: a row block's entries fall into n
// column runs of a few entries, every store leaves L2 as a partial-line write of its own, and 100M
// ratings x 17,770 columns take 5.6 ms for 0.8 GB of output.  So, where the workspace can hold the
// entries once (rx_layout), they are sorted by column digit, at most 8 bits a pass, lowest first: two
// passes for n <= 65,536, three up to 2^24 columns, one for n <= 256.  The bits are dealt evenly, the
// first pass getting the fewest: its digits are the most evenly spread, so its runs are the shortest
// (a tile's entries over its digits).  A pass cuts the entries into
// kRxBlocks equal ranges, counts digits per range (k_rx_count), makes the counts offsets
// (k_rx_offsets) and moves the entries (k_rx_move): tiles of 4,096 entries are ranked by digit
// (stable: a wave ranks 64 consecutive entries by ballots), put in order in LDS and written out in
// runs of at least 16 entries per digit on average.  From the second pass on, k_rx_count also counts every
// combination of the digit with the lower ones, the last of them being the columns' counts: the
// entries are already sorted by the lower digits, so it counts one lower value's stretch at a time
// in LDS and adds it to the global counts once.
// Movie matrix: 6.4 -> 2.0 ms for the whole transpose; 250,000 x 625,000 with 62.5M ratings, whose
// counters do not fit in LDS: 9.5 -> 1.8 ms.  (8 bits in the first pass: 2.06 and 2.04 ms; 768 blocks
// instead of 1,536: 2.44 and 2.32 ms.)
constexpr int kRxThreads = 256;
constexpr int kRxWaves = kRxThreads / kWave;
constexpr int kRxPer = 16;                                // entries per thread and tile
constexpr int kRxTile = kRxThreads * kRxPer;
constexpr int kRxDigits = 256;
constexpr int kRxBlocks = 1536;   // twice what is resident (three blocks of 53 KB of LDS per CU)
constexpr int64_t kRxMaxCols = 1 << 24;

// The entries of a pass.  From the CSR (key null): colidx, vals and the row of each position;
// between passes: row, value and the column bits above the digits already sorted by.
struct RxSrc {
    const int64_t* rowptr;
    int64_t m;
    const int32_t* colidx;   // first pass
    const float* vals;
    const uint32_t* row;     // later passes
    const float* val;
    const uint16_t* key;
};

// Sum of the counts before and the sum of all of counts[0, 256), one per thread.
__device__ __forceinline__ int rx_scan256(int x, int* sh, int* total) {
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int inc = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o);
        if (lane >= o) inc += y;
    }
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int base = 0;
    for (int i = 0; i < w; ++i) base += sh[i];
    *total = sh[0] + sh[1] + sh[2] + sh[3];
    __syncthreads();
    return base + inc - x;
}

// Entries [lo, hi) of block b's range of `count` entries.
__device__ __forceinline__ void rx_range(int count, int b, int& lo, int& hi) {
    lo = (int)((int64_t)count * b / kRxBlocks);
    hi = (int)((int64_t)count * (b + 1) / kRxBlocks);
}

// First pass: digit counts of the CSR's ranges (columns outside [0, n) left out), hist[d][b].
__global__ __launch_bounds__(kRxThreads) void k_rx_count_first(
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ colidx, int64_t m, int n,
    int64_t cap, int width, int* __restrict__ hist) {
    if (rowptr[m] > cap) return;
    __shared__ int h[kRxDigits];
    const int mask = (1 << width) - 1;   // a digit of `width` bits
    const int t = threadIdx.x, b = blockIdx.x;
    h[t] = 0;
    __syncthreads();
    int lo, hi;
    rx_range((int)rowptr[m], b, lo, hi);
    for (int k0 = lo; k0 < hi; k0 += 4 * kRxThreads) {
        int v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + j * kRxThreads + t;
            v[j] = k < hi ? colidx[k] : -1;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (v[j] >= 0 && v[j] < n) atomicAdd(&h[v[j] & mask], 1);
    }
    lds_atomics_done();
    __syncthreads();
    hist[t * kRxBlocks + b] = h[t];
}

// Later passes: digit counts of the ranges, and counts[digit << bits | lower] for every lower
// value, whose entries are [starts[lower], starts[lower + 1]).  OUT is int (the starts' counts of
// the next pass) or unsigned long long (the columns' counts, in colptr).
template <class OUT>
__global__ __launch_bounds__(kRxThreads) void k_rx_count(const int64_t* __restrict__ rowptr,
                                                         int64_t m, int64_t cap,
                                                         const uint16_t* __restrict__ key,
                                                         const int* __restrict__ starts, int bits,
                                                         int width, int64_t limit,
                                                         int* __restrict__ hist,
                                                         OUT* __restrict__ counts) {
    if (rowptr[m] > cap) return;
    __shared__ int h[kRxDigits];
    const int t = threadIdx.x, b = blockIdx.x, mask = (1 << width) - 1;
    int lo, hi;
    rx_range(starts[1 << bits], b, lo, hi);
    // the last lower value from `low` on that starts at or before entry k: the one that holds it
    const auto holder = [&](int low, int k) {
        int top = (1 << bits) - 1;
        while (low < top) {
            const int mid = (low + top + 1) >> 1;
            if (starts[mid] <= k) low = mid; else top = mid - 1;
        }
        return low;
    };
    int all = 0, low = holder(0, lo);
    h[t] = 0;
    __syncthreads();
    for (int k = lo; k < hi; ++low) {
        if (starts[low + 1] <= k) low = holder(low, k);   // past lower values without entries
        const int next = starts[low + 1], end = next < hi ? next : hi;
        for (int k0 = k; k0 < end; k0 += 4 * kRxThreads) {
            int v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = k0 + j * kRxThreads + t;
                v[j] = i < end ? (int)key[i] : -1;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (v[j] >= 0) atomicAdd(&h[v[j] & mask], 1);
        }
        lds_atomics_done();
        __syncthreads();
        const int c = h[t];
        h[t] = 0;
        all += c;
        const int64_t at = ((int64_t)t << bits) | low;
        if (c && at < limit) atomicAdd(&counts[at], (OUT)c);
        __syncthreads();
        k = end;
    }
    hist[t * kRxBlocks + b] = all;
}

// Per digit: its ranges' counts -> offsets within the digit, and the digit's total (after the
// first pass also colptr[d] when the digit is the whole column).
__global__ __launch_bounds__(kRxThreads) void k_rx_offsets(const int64_t* __restrict__ rowptr,
                                                           int64_t m, int64_t cap,
                                                           int* __restrict__ hist,
                                                           int* __restrict__ totals,
                                                           int64_t* __restrict__ colptr, int n) {
    if (rowptr[m] > cap) return;
    __shared__ int sh[kRxWaves];
    const int d = blockIdx.x, t = threadIdx.x;
    constexpr int kPer = kRxBlocks / kRxThreads;
    int* h = hist + d * kRxBlocks + t * kPer;
    int v[kPer], sum = 0, total;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        v[j] = h[j];
        sum += v[j];
    }
    int run = rx_scan256(sum, sh, &total);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        h[j] = run;
        run += v[j];
    }
    if (t == 0) {
        totals[d] = total;
        if (colptr && d < n) colptr[d] = total;
    }
}

// starts[0, 2^bits] from counts (one workgroup).
__global__ __launch_bounds__(kRxThreads) void k_rx_starts(const int64_t* __restrict__ rowptr,
                                                          int64_t m, int64_t cap,
                                                          const int* __restrict__ counts, int bits,
                                                          int* __restrict__ starts) {
    if (rowptr[m] > cap) return;
    __shared__ int sh[kRxWaves];
    const int t = threadIdx.x, size = 1 << bits;
    int carry = 0;
    for (int base = 0; base < size; base += kRxThreads * 16) {
        int v[16], sum = 0, total;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int i = base + t * 16 + j;
            v[j] = i < size ? counts[i] : 0;
            sum += v[j];
        }
        int run = carry + rx_scan256(sum, sh, &total);
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int i = base + t * 16 + j;
            if (i < size) starts[i] = run;
            run += v[j];
        }
        carry += total;
    }
    if (t == 0) starts[size] = carry;
}

// Move a pass's entries to their places.  FIRST: from the CSR.  LAST: no key is written.
template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kRxThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_rx_move(RxSrc in, int n, int64_t cap, int width,
                                                        const int* __restrict__ hist,
                                                        const int* __restrict__ totals,
                                                        uint32_t* __restrict__ row_out,
                                                        float* __restrict__ val_out,
                                                        uint16_t* __restrict__ key_out) {
    if (in.rowptr[in.m] > cap) return;
    __shared__ uint32_t srow[kRxTile];
    __shared__ float sval[kRxTile];
    __shared__ uint32_t skey[kRxTile];   // first the row marks of the tile, then the keys in order
    __shared__ int wcnt[kRxWaves][kRxDigits];   // counts, then places in the tile's order
    __shared__ int shift[kRxDigits];            // from a place in the tile's order to the output
    __shared__ int sh[kRxWaves];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, b = blockIdx.x;
    const uint32_t mask = (1u << width) - 1;
    int count;
    // where this block's next entry of digit t goes
    int dest = rx_scan256(totals[t], sh, &count) + hist[t * kRxBlocks + b];
    if (FIRST) count = (int)in.rowptr[in.m];
    int lo, hi;
    rx_range(count, b, lo, hi);
    int64_t u = 0;   // FIRST: row of the tile's first entry
    if (FIRST && lo < hi) {
        int64_t a = 0, z = in.m - 1;   // largest row that starts at or before lo
        while (a < z) {
            const int64_t mid = (a + z + 1) >> 1;
            if (in.rowptr[mid] <= lo) a = mid; else z = mid - 1;
        }
        u = a;
    }
    for (int t0 = lo; t0 < hi; t0 += kRxTile) {
        const int t1 = t0 + kRxTile < hi ? t0 + kRxTile : hi;
        const int wbase = t0 + w * kRxPer * kWave;   // this wave's entries of the tile
        uint32_t key[kRxPer], row[kRxPer];
        float val[kRxPer];
#pragma unroll
        for (int j = 0; j < kRxPer; ++j) {
            const int k = wbase + j * kWave + lane;
            key[j] = 0xFFFFFFFFu;   // not an entry
            if (k < t1) {
                if (FIRST) {
                    const int c = in.colidx[k];
                    if (c >= 0 && c < n) key[j] = (uint32_t)c;
                    val[j] = in.vals[k];
                } else {
                    key[j] = in.key[k];
                    val[j] = in.val[k];
                    row[j] = in.row[k];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kRxWaves; ++i) wcnt[i][t] = 0;
        if (FIRST) {
            // mark where rows start in the tile (the last one of several that start together), by
            // their distance from u; the last mark at or before an entry is its row
#pragma unroll
            for (int j = 0; j < kRxPer; ++j) skey[j * kRxThreads + t] = 0;
            __syncthreads();
            int64_t passed = 0;   // rows after u that start before t1
            for (int64_t r0 = u + 1;; r0 += kRxThreads) {
                const int64_t r = r0 + t;
                const int64_t at = r < in.m ? in.rowptr[r] : (int64_t)t1;
                const bool inside = at < t1;
                if (inside) atomicMax(&skey[at - t0], (uint32_t)(r - u));
                lds_atomics_done();
                const int c = __syncthreads_count(inside);
                passed += c;
                if (c < kRxThreads) break;
            }
            uint32_t last = 0;   // the wave's last mark so far (marks grow with their place)
#pragma unroll
            for (int j = 0; j < kRxPer; ++j) {
                const uint32_t x = skey[w * kRxPer * kWave + j * kWave + lane];
                const uint64_t marks = __ballot(x != 0);
                const uint64_t upto = marks & (~0ull >> (63 - lane));
                const uint32_t own = (uint32_t)__shfl((int)x, upto ? 63 - __builtin_clzll(upto) : 0);
                row[j] = upto ? own : last;
                if (marks)
                    last = (uint32_t)__builtin_amdgcn_readlane((int)x, 63 - __builtin_clzll(marks));
            }
            if (lane == 0) sh[w] = (int)last;
            __syncthreads();
            uint32_t before = 0;   // the earlier waves' last mark
            for (int i = 0; i < w; ++i) before = max(before, (uint32_t)sh[i]);
#pragma unroll
            for (int j = 0; j < kRxPer; ++j) row[j] = (uint32_t)u + max(row[j], before);
            u += passed;
        }
        __syncthreads();
        // rank by digit within the wave's entries
        int rank[kRxPer];
#pragma unroll
        for (int j = 0; j < kRxPer; ++j) {
            const bool live = key[j] != 0xFFFFFFFFu;
            const uint32_t d = key[j] & mask;
            uint64_t same = __ballot(live);
#pragma unroll
            for (int bit = 0; bit < 8; ++bit) {
                const uint64_t has = __ballot((d >> bit) & 1);
                same &= ((d >> bit) & 1) ? has : ~has;
            }
            const int before = __popcll(same & ((1ull << lane) - 1));
            int old = 0;
            if (live && before == 0) old = atomicAdd(&wcnt[w][d], __popcll(same));
            rank[j] = before + __shfl(old, live ? __builtin_ctzll(same) : lane);
        }
        lds_atomics_done();
        __syncthreads();
        int c[kRxWaves], sum = 0, tile;   // thread t: digit t
#pragma unroll
        for (int i = 0; i < kRxWaves; ++i) {
            c[i] = wcnt[i][t];
            sum += c[i];
        }
        int place = rx_scan256(sum, sh, &tile);
        shift[t] = dest - place;
        dest += sum;
#pragma unroll
        for (int i = 0; i < kRxWaves; ++i) {
            wcnt[i][t] = place;
            place += c[i];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kRxPer; ++j) {
            if (key[j] != 0xFFFFFFFFu) {
                const uint32_t d = key[j] & mask;
                const int at = wcnt[w][d] + rank[j];
                srow[at] = row[j];
                sval[at] = val[j];
                skey[at] = key[j];
            }
        }
        __syncthreads();
        for (int i = t; i < tile; i += kRxThreads) {
            const uint32_t k = skey[i];
            const int to = i + shift[k & mask];
            row_out[to] = srow[i];
            val_out[to] = sval[i];
            if (!LAST) key_out[to] = (uint16_t)(k >> width);
        }
        __syncthreads();
    }
}

// --------------------------------------------------------------------- host side ---------

struct Layout {
    size_t status, bounds, rmse, slots, wave_slots, total;
};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// waves[nb][last] = W for nb column blocks and a form of the last one (0 where f has no such form);
// the slot region holds 2 C partial accumulators,
// C = chunks_of(W), and the wave-slot region one more per wave (the second summation level of
// long pieces)
Layout make_layout(const int (*waves)[kLastForms], int nb_max, int cus) {
    int c_cap = 1;
    size_t slot_bytes = 0, wave_bytes = 0;
    for (int nb = 1; nb <= nb_max; ++nb) {
        int w = 0;
        for (int last = 0; last < kLastForms; ++last)
            if (waves[nb][last] > w) w = waves[nb][last];
        const int C = chunks_of(w);
        if (C > c_cap) c_cap = C;
        const size_t sb = sizeof(float) * (size_t)slot_floats(nb) * 2 * (size_t)C;
        if (sb > slot_bytes) slot_bytes = sb;
        const size_t wb = sizeof(float) * (size_t)slot_floats(nb) * (size_t)w;
        if (wb > wave_bytes) wave_bytes = wb;
    }
    Layout L;
    size_t off = 0;
    // non-SPD counter at 0, RMSE chunk counter at 128, flag of rows set aside at 192, the half-sweep's
    // chunk counters from 256 on
    L.status = off; off = align256(off + 256 + sizeof(unsigned) * kStripes * kStripeWords);
    L.bounds = off; off = align256(off + sizeof(int64_t) * 2 * (size_t)(c_cap + 1));
    L.rmse = off;   off = align256(off + sizeof(double) * (size_t)cus * kRmseWavesPerCU);
    L.slots = off;  off = align256(off + slot_bytes);
    L.wave_slots = off; off = align256(off + wave_bytes);
    L.total = off;
    return L;
}

// Whether some f <= ALS_F_MAX with nb column blocks runs with this form of the last one (ordinary
// tiles can be asked for at every f).
constexpr bool last_exists(int nb, int last) {
    if (last == kLastTiles) return true;
    return last == kLastRating ? nb >= 2 : 16 * (nb - 1) + 1 <= ALS_F_MAX;
}

// Resident waves per CU of both gather forms (the partition is shared, so every wave of either
// form is resident at once).
template <int NB, int LAST>
int occupancy_waves(int* waves) {
    *waves = 0;
    if constexpr (last_exists(NB, LAST)) {
        int blocks = kMaxWavesPerCU;
        const void* forms[] = {(const void*)k_herm_solve<NB, kFormBuffer, LAST, false>,
                               (const void*)k_herm_solve<NB, kFormGlobal, LAST, false>,
                               (const void*)k_herm_solve<NB, kFormBuffer, LAST, true>,
                               (const void*)k_herm_solve<NB, kFormGlobal, LAST, true>};
        for (const void* k : forms) {
            int b = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k, kWave, 0) != hipSuccess)
                return -1;
            if (b < blocks) blocks = b;
        }
        if (blocks < 1) blocks = 1;
        *waves = blocks;
    }
    return 0;
}

template <int NB>
int occupancy_forms(int* waves) {
    if (occupancy_waves<NB, kLastTiles>(waves + kLastTiles) != 0 ||
        occupancy_waves<NB, kLastPacked>(waves + kLastPacked) != 0)
        return -1;
    return occupancy_waves<NB, kLastRating>(waves + kLastRating);
}

// Launch the RMSE partials kernel over C = cus * kRmseWavesPerCU chunks (the partials buffer
// holds that many) with as many resident waves as fit, at most `cap_per_cu` per CU if that is
// positive.  A grid of fewer waves than chunks claims them: its counter is reset first, on the
// same stream.
template <int NB, bool BUF>
hipError_t rmse_rows_launch(int cus, int cap_per_cu, hipStream_t st, const int64_t* rowptr,
                            const int32_t* colidx, const float* vals, int64_t m, int64_t n,
                            int f, const float* x, const float* theta, double* part,
                            unsigned* claim, int C) {
    int b = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &b, (const void*)k_rmse_rows<NB, BUF>, kWave, 0);
    if (e != hipSuccess) return e;
    b = b < 1 ? 1 : (b > kRmseWavesPerCU ? kRmseWavesPerCU : b);
    if (cap_per_cu > 0 && b > cap_per_cu) b = cap_per_cu;
    if (cus * b < C)
        hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, st, (unsigned long long*)claim);
    hipLaunchKernelGGL((k_rmse_rows<NB, BUF>), dim3(cus * b), dim3(kWave), 0, st, rowptr,
                       colidx, vals, m, n, f, x, theta, C, part, claim);
    return hipGetLastError();
}

int waves_per_cu(int nb, int* w) {
    switch (nb) {
        case 1: return occupancy_forms<1>(w);
        case 2: return occupancy_forms<2>(w);
        case 3: return occupancy_forms<3>(w);
        case 4: return occupancy_forms<4>(w);
        case 5: return occupancy_forms<5>(w);
        case 6: return occupancy_forms<6>(w);
        case 7: return occupancy_forms<7>(w);
        case 8: return occupancy_forms<8>(w);
        case 9: return occupancy_forms<9>(w);
        default: return -1;
    }
}

template <int NB>
int staged_occupancy(int cus, int* waves) {
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &b, (const void*)k_herm_solve<NB, kFormStaged, kLastTiles, true>, kWave, 0) !=
        hipSuccess)
        return -1;
    int b2 = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &b2, (const void*)k_herm_solve<NB, kFormStaged, kLastTiles, false>, kWave, 0) !=
        hipSuccess)
        return -1;
    if (b2 < b) b = b2;
    if (b < 1) b = 1;
    if (b > kMaxWavesPerCU) b = kMaxWavesPerCU;
    *waves = b * cus;
    return 0;
}

int staged_waves_for_nb(int nb, int cus, int* w) {
    switch (nb) {
        case 1: return staged_occupancy<1>(cus, w);
        case 2: return staged_occupancy<2>(cus, w);
        case 3: return staged_occupancy<3>(cus, w);
        case 4: return staged_occupancy<4>(cus, w);
        case 5: return staged_occupancy<5>(cus, w);
        case 6: return staged_occupancy<6>(cus, w);
        case 7: return staged_occupancy<7>(cus, w);
        case 8: return staged_occupancy<8>(cus, w);
        case 9: return staged_occupancy<9>(cus, w);
        default: return -1;
    }
}

int nb_of(int f) { return f / 16 + 1; }   // blocks of 16 covering the augmented f + 1

// Solve cost of one row in c_nnz units: per 16-column block about 2,500 cycles of factor and
// inverse on the vector ALU plus the panel and trailing-update MFMAs (32 cycles each); the
// vector part overlaps other waves' matrix work, so half of the total is charged.  Tunable
// through ALS_ROW_COST (entries per row).
int64_t row_cost(int f) {
    const char* env = getenv("ALS_ROW_COST");
    if (env && atoll(env) > 0) return atoll(env) * kCostPerEntry;
    const int nb = nb_of(f);
    const double mfma_cycles_per_entry = 8.0 * ntiles(nb);
    double mfmas = 0;
    for (int K = 0; K < nb; ++K) mfmas += 4.0 * ((nb - K - 1) + (nb - K - 1) * (nb - K) / 2.0);
    const double solve_cycles = 2500.0 * nb + 32.0 * mfmas;
    double entries = 0.5 * solve_cycles / mfma_cycles_per_entry;
    if (entries < 1.0) entries = 1.0;
    return (int64_t)(entries * kCostPerEntry);
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

}  // namespace

struct als_ctx {
    int device;
    int cus;
    int f_max;
    int nb_max;
    int w_cap;
    int waves[kMaxNB + 1][kLastForms];
    unsigned char* ws;
    size_t ws_bytes;
    Layout lay;
    int last_hip;
    hipEvent_t* prof_ev;   // 4 events per profiled half-sweep, or null
    int prof_cap;
    int prof_count;
    bool global_gather;    // use the 64-bit-load gather for every size (ALS_GATHER=global)
    bool staged_gather;    // stage theta through LDS (ALS_GATHER=lds; ablation)
    bool tile_last_block;  // 16x16 tiles for the last block column always (ALS_LAST_BLOCK=tiles)
    int rmse_waves_per_simd;   // cap on resident RMSE waves per SIMD (0 = as many as fit)
    int part_groups;           // pipeline groups per part of a long piece (a power of two)
    size_t lds_per_block;      // the device's LDS bytes per workgroup
};

namespace {

int fail_hip(als_ctx* ctx, hipError_t e) {
    if (ctx) ctx->last_hip = (int)e;
    return ALS_ERR_HIP;
}

struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        ok = (prev == dev) || hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

// What a device is and how many waves of each kernel fit it: asked for once per device and process
// (with the queries in every call, als_workspace_bytes and als_init took 46 us together, now 28).  Column-block counts are added as they are needed.
struct DeviceInfo {
    std::mutex mu;
    bool known = false;
    int cus = 0;
    size_t lds_per_block = 0;
    int nb_known = 0;                            // per_cu holds 1..nb_known
    int per_cu[kMaxNB + 1][kLastForms] = {{0}};  // resident waves per CU
};
constexpr int kMaxDevices = 64;
DeviceInfo g_device[kMaxDevices];

int query_device(int device, int f_max, int* cus, int (*waves)[kLastForms], int* w_cap,
                 size_t* lds_per_block = nullptr) {
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n || device >= kMaxDevices)
        return ALS_ERR_DEVICE;
    DeviceInfo& d = g_device[device];
    std::lock_guard<std::mutex> lock(d.mu);
    DeviceGuard guard(device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    if (!d.known) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, device) != hipSuccess) return ALS_ERR_DEVICE;
        if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return ALS_ERR_DEVICE;
        d.cus = prop.multiProcessorCount;
        d.lds_per_block = prop.sharedMemPerBlock;
        d.known = true;
    }
    for (; d.nb_known < nb_of(f_max); ++d.nb_known)
        if (waves_per_cu(d.nb_known + 1, d.per_cu[d.nb_known + 1]) != 0) return ALS_ERR_HIP;
    *cus = d.cus;
    if (lds_per_block) *lds_per_block = d.lds_per_block;
    const char* env = getenv("ALS_WAVES_PER_CU");
    const int limit = env && atoi(env) > 0 ? atoi(env) : kMaxWavesPerCU;
    *w_cap = 1;
    for (int nb = 1; nb <= nb_of(f_max); ++nb)
        for (int last = 0; last < kLastForms; ++last) {
            const int w = d.per_cu[nb][last];
            waves[nb][last] = (w < limit ? w : limit) * d.cus;
            if (waves[nb][last] > *w_cap) *w_cap = waves[nb][last];
        }
    return ALS_OK;
}

// theta sizes (bytes) served by the buffer-load gather: offsets past the end, plus a padding
// lane's offset, must stay below 2^32
constexpr uint64_t kBufferGatherMax = 0x7FFFF000ull;

// The staged gather (an ablation form) reads whole 16-byte groups of a row through one buffer
// descriptor.
bool staged_supported(int64_t n, int f) {
    return f % 4 == 0 && (uint64_t)n * (uint64_t)f * sizeof(float) <= kBufferGatherMax;
}

// The form of the last block column that a half-sweep of this context uses at f.
int form_of(const als_ctx* ctx, int f) {
    return ctx->staged_gather || ctx->tile_last_block ? kLastTiles : last_form(f);
}

struct HermArgs {
    const int64_t* rowptr;
    const int32_t* colidx;
    const float* vals;
    const float* theta;
    int64_t m, n;
    int f;
    float lambda;
    int C;
    const int64_t* bounds;
    float* x;
    float* slots;
    float* wslots;
    int part_mask;
    int64_t c_row;
    unsigned long long* nonspd;
    unsigned* chunk_ctr;
    unsigned* set_aside;
};

// A row has at most n entries (its columns are distinct), so with n no longer than a part no piece
// is.  Beyond that both instantiations are launched; the kernels pick the one that runs from
// rowptr[m] on the device (no host synchronisation), the other returns at once (about 5 us).
template <int NB, int BUF, int LAST>
void launch_herm(int W, hipStream_t st, const HermArgs& a) {
    hipLaunchKernelGGL((k_herm_solve<NB, BUF, LAST, false>), dim3(W), dim3(kWave), 0, st,
                       a.rowptr, a.colidx, a.vals, a.theta, a.m, a.n, a.f, a.lambda, a.C,
                       a.bounds, a.x, a.slots, a.wslots, a.part_mask, a.c_row, a.nonspd,
                       a.chunk_ctr, a.set_aside);
    if (a.n <= (int64_t)kGroupEntries * (a.part_mask + 1)) return;
    hipLaunchKernelGGL((k_herm_solve<NB, BUF, LAST, true>), dim3(W), dim3(kWave), 0, st,
                       a.rowptr, a.colidx, a.vals, a.theta, a.m, a.n, a.f, a.lambda, a.C,
                       a.bounds, a.x, a.slots, a.wslots, a.part_mask, a.c_row, a.nonspd,
                       a.chunk_ctr, a.set_aside);
}

// fn with the form of the last block column as a constant.
template <int NB, class Fn>
void with_last_form(int last, Fn&& fn) {
    if (last == kLastTiles) fn(std::integral_constant<int, kLastTiles>{});
    if constexpr (last_exists(NB, kLastPacked)) {
        if (last == kLastPacked) fn(std::integral_constant<int, kLastPacked>{});
    }
    if constexpr (last_exists(NB, kLastRating)) {
        if (last == kLastRating) fn(std::integral_constant<int, kLastRating>{});
    }
}

template <int NB>
void launch_sweep(als_ctx* ctx, const int64_t* rowptr, const int32_t* colidx, const float* vals,
                  int64_t m, int64_t n, int f, float lambda, const float* theta, float* x,
                  hipStream_t st, int W) {
    int64_t* bounds = (int64_t*)(ctx->ws + ctx->lay.bounds);
    float* slots = (float*)(ctx->ws + ctx->lay.slots);
    float* wslots = (float*)(ctx->ws + ctx->lay.wave_slots);
    const int part_mask = ctx->part_groups - 1;
    auto* nonspd = (unsigned long long*)(ctx->ws + ctx->lay.status);
    auto* chunk_ctr = (unsigned*)(ctx->ws + ctx->lay.status + 256);
    auto* set_aside = (unsigned*)(ctx->ws + ctx->lay.status + 192);
    const int C = chunks_of(W);
    hipEvent_t* ev = nullptr;
    if (ctx->prof_ev && ctx->prof_count < ctx->prof_cap) ev = ctx->prof_ev + 4 * ctx->prof_count++;
    if (ev) (void)hipEventRecord(ev[0], st);
    hipLaunchKernelGGL(k_plan, dim3((C + 1 + 63) / 64), dim3(64), 0, st, rowptr, m, W, C,
                       (int64_t)kCostPerEntry, row_cost(f), (int64_t)kSnap, bounds, chunk_ctr,
                       set_aside);
    if (ev) (void)hipEventRecord(ev[1], st);
    const HermArgs a{rowptr, colidx, vals, theta, m, n, f, lambda, C, bounds, x, slots, wslots,
                     part_mask, row_cost(f), nonspd, chunk_ctr, set_aside};
    const bool buf = !ctx->global_gather &&
                     (uint64_t)n * (uint64_t)f * sizeof(float) <= kBufferGatherMax;
    if (ctx->staged_gather) {   // f % 4 == 0 and theta below 2 GiB (checked by the caller)
        launch_herm<NB, kFormStaged, kLastTiles>(W, st, a);
    } else {
        with_last_form<NB>(form_of(ctx, f), [&](auto last) {
            if (buf) launch_herm<NB, kFormBuffer, last.value>(W, st, a);
            else launch_herm<NB, kFormGlobal, last.value>(W, st, a);
        });
    }
    if (ev) (void)hipEventRecord(ev[2], st);
    if (C > 1) {
        const int grid = C - 1 < kReduceWaves ? C - 1 : kReduceWaves;
        hipLaunchKernelGGL(k_reduce_groups<NB>, dim3(grid), dim3(kWave), 0, st, rowptr, m, C,
                           bounds, slots);
        hipLaunchKernelGGL(k_reduce_solve<NB>, dim3(grid), dim3(kWave), 0, st, rowptr, colidx, vals,
                           theta, m, C, f, lambda, bounds, x, slots, nonspd, set_aside);
    }
    if (ev) (void)hipEventRecord(ev[3], st);
}

// The gather form k_herm_solve would use for this call (buffer loads or 64-bit loads; the form of the
// last block column), run by k_gather_dump on row u.
template <int NB>
void launch_dump(als_ctx* ctx, const int64_t* rowptr, const int32_t* colidx, const float* vals,
                 int64_t n, int f, const float* theta, int64_t u, float* out, int64_t limit,
                 hipStream_t st) {
    const bool buf = !ctx->global_gather &&
                     (uint64_t)n * (uint64_t)f * sizeof(float) <= kBufferGatherMax;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kWave), 0, st, rowptr, colidx, vals, theta, n, f,
                           u, out, limit);
    };
    if (ctx->staged_gather) {
        launch(k_gather_dump<NB, kFormStaged, kLastTiles>);
    } else {
        with_last_form<NB>(form_of(ctx, f), [&](auto last) {
            if (buf) launch(k_gather_dump<NB, kFormBuffer, last.value>);
            else launch(k_gather_dump<NB, kFormGlobal, last.value>);
        });
    }
}

// ---------------------------------------------------------- fixed scratch (no workspace) ---

// als_rmse_noalloc's scratch: the claim counter (at 0) and one fp64 partial per RMSE chunk (at
// 256), for devices of up to kNoAllocMaxCUs compute units.  Each device holds its own copy of
// the array; host code reaches a device's copy only through the address hipGetSymbolAddress
// returns with that device current (the array's name is a host-side stand-in).
constexpr int kNoAllocMaxCUs = 320;
constexpr size_t kNoAllocPartials = 256;
constexpr size_t kNoAllocScratchBytes =
    kNoAllocPartials + sizeof(double) * (size_t)kNoAllocMaxCUs * kRmseWavesPerCU;
struct NoAllocDevice {
    std::once_flag once;
    int rc = ALS_ERR_DEVICE;
    unsigned char* ptr = nullptr;   // this device's copy of the scratch array
    int cus = 0;
};
NoAllocDevice g_noalloc[kMaxDevices];

}  // namespace

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

// Once per device, with that device current: its compute units and the device address of its
// copy of `scratch`.  Called by als_init and by the first als_rmse_noalloc on a device.
int noalloc_setup(int device) {
    if (device < 0 || device >= kMaxDevices) return ALS_ERR_DEVICE;
    NoAllocDevice& d = g_noalloc[device];
    std::call_once(d.once, [&d, device]() {
        int n = 0;
        if (hipGetDeviceCount(&n) != hipSuccess || device >= n) return;
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, device) != hipSuccess) return;
        if (strncmp(prop.gcnArchName, "gfx950", 6) != 0) return;
        DeviceGuard guard(device);
        if (!guard.ok) return;
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            d.rc = ALS_ERR_HIP;
            return;
        }
        d.ptr = (unsigned char*)ptr;
        d.cus = prop.multiProcessorCount;
        d.rc = ALS_OK;
    });
    return d.rc;
}

int rmse_check(const int64_t* rowptr, const int32_t* colidx, const float* vals, int64_t m,
               int64_t n, int32_t f, const float* x, const float* theta, const double* rmse_out) {
    if (f < 1 || f > ALS_F_MAX) return ALS_ERR_UNSUPPORTED_F;
    if (m < 0 || n < 0 || !rowptr || !rmse_out) return ALS_ERR_INVALID_ARG;
    if (m > 0 && (!x || (n > 0 && (!colidx || !vals || !theta)))) return ALS_ERR_INVALID_ARG;
    if (!aligned(rowptr, 8) || !aligned(colidx, 4) || !aligned(vals, 4) || !aligned(x, 4) ||
        !aligned(theta, 4) || !aligned(rmse_out, 8))
        return ALS_ERR_ALIGN;
    return ALS_OK;
}

// The RMSE's two kernels on `st`: partials over C = cus * kRmseWavesPerCU fixed chunks (at most
// cap_per_cu resident waves per CU if positive), then their fixed-order sum.  part holds C
// doubles; claim is the chunk counter (reset here by a kernel).
hipError_t rmse_launch(int cus, int cap_per_cu, bool force_global, hipStream_t st,
                       const int64_t* rowptr, const int32_t* colidx, const float* vals, int64_t m,
                       int64_t n, int f, const float* x, const float* theta, double* part,
                       unsigned* claim, double* rmse_out) {
    const int C = cus * kRmseWavesPerCU;
    if (m > 0) {
        const bool buf =
            !force_global && (uint64_t)n * (uint64_t)f * sizeof(float) <= kBufferGatherMax;
        hipError_t le = hipSuccess;
#define ALS_RMSE_ARGS cus, cap_per_cu, st, rowptr, colidx, vals, m, n, f, x, theta, part, claim, C
        switch (f / 16 + 1) {
#define ALS_RMSE_CASE(NB)                                                           \
            case NB:                                                                \
                le = buf ? rmse_rows_launch<NB, true>(ALS_RMSE_ARGS)                \
                         : rmse_rows_launch<NB, false>(ALS_RMSE_ARGS);              \
                break;
            ALS_RMSE_CASE(1) ALS_RMSE_CASE(2) ALS_RMSE_CASE(3) ALS_RMSE_CASE(4) ALS_RMSE_CASE(5)
            ALS_RMSE_CASE(6) ALS_RMSE_CASE(7) ALS_RMSE_CASE(8) ALS_RMSE_CASE(9)
#undef ALS_RMSE_CASE
#undef ALS_RMSE_ARGS
            default: return hipErrorInvalidValue;
        }
        if (le != hipSuccess) return le;
    }
    hipLaunchKernelGGL(k_rmse_final, dim3(1), dim3(kFinalThreads), 0, st, rowptr, m, m > 0 ? C : 0, part,
                       rmse_out);
    return hipGetLastError();
}

// The radix transpose's share of the workspace.
struct RxSpace {
    int passes;            // 1..3
    int width[3];          // bits of each pass's digit
    int *hist, *totals, *counts, *starts;
    uint32_t* row;         // entries between passes
    float* val;
    uint16_t *key, *key2;  // key2: after the first of three passes (row and value in the outputs)
};

// Lay it out in `bytes` at p (256-byte aligned); returns how many entries it holds (0: the sort
// cannot run).
int64_t rx_layout(unsigned char* p, size_t bytes, int64_t n, RxSpace* rx) {
    if (n > kRxMaxCols) return 0;
    int bits = 1;
    while (((int64_t)1 << bits) < n) ++bits;
    rx->passes = (bits + 7) / 8;
    for (int i = 0; i < rx->passes; ++i)
        rx->width[i] = bits / rx->passes + (i >= rx->passes - bits % rx->passes ? 1 : 0);
    size_t off = 0;
    const auto take = [&](size_t b) {
        unsigned char* at = p + off;
        off = align256(off + b);
        return at;
    };
    rx->hist = (int*)take(sizeof(int) * kRxDigits * kRxBlocks);
    rx->totals = (int*)take(sizeof(int) * kRxDigits);
    rx->counts = (int*)take(sizeof(int) << 16);
    rx->starts = (int*)take(sizeof(int) * ((1 << 16) + 1));
    if (rx->passes == 1) return off <= bytes ? INT32_MAX / 2 : 0;
    const size_t each = sizeof(uint32_t) + sizeof(float) +
                        (rx->passes - 1) * sizeof(uint16_t);
    const size_t slack = 4 * 256;   // alignment of the arrays below
    if (bytes < off + slack + each) return 0;
    int64_t cap = (int64_t)((bytes - off - slack) / each);
    if (cap > INT32_MAX / 2) cap = INT32_MAX / 2;
    rx->row = (uint32_t*)take(sizeof(uint32_t) * (size_t)cap);
    rx->val = (float*)take(sizeof(float) * (size_t)cap);
    rx->key = (uint16_t*)take(sizeof(uint16_t) * (size_t)cap);
    rx->key2 = (uint16_t*)take(rx->passes == 3 ? sizeof(uint16_t) * (size_t)cap : 0);
    return cap;
}

// The passes (see k_rx_count_first); colptr is zeroed and left with the columns' counts.
void rx_launch(const RxSpace& rx, int64_t cap, hipStream_t st, const int64_t* rowptr,
               const int32_t* colidx, const float* vals, int64_t m, int64_t n, int64_t* colptr,
               uint32_t* rowidx, float* vals_t) {
    const dim3 grid(kRxBlocks), block(kRxThreads), digits(kRxDigits);
    auto* columns = (unsigned long long*)colptr;
    const RxSrc csr{rowptr, m, colidx, vals, nullptr, nullptr, nullptr};
    const RxSrc out{rowptr, m, nullptr, nullptr, rowidx, vals_t, rx.key2};
    const RxSrc mid{rowptr, m, nullptr, nullptr, rx.row, rx.val, rx.key};
    const int w0 = rx.width[0], w1 = rx.width[1], w2 = rx.width[2];
    hipLaunchKernelGGL(k_rx_count_first, grid, block, 0, st, rowptr, colidx, m, (int)n, cap, w0,
                       rx.hist);
    hipLaunchKernelGGL(k_rx_offsets, digits, block, 0, st, rowptr, m, cap, rx.hist, rx.totals,
                       rx.passes == 1 ? colptr : nullptr, (int)n);
    if (rx.passes == 1) {
        hipLaunchKernelGGL((k_rx_move<true, true>), grid, block, 0, st, csr, (int)n, cap, w0,
                           rx.hist, rx.totals, rowidx, vals_t, nullptr);
        return;
    }
    hipLaunchKernelGGL(k_rx_starts, dim3(1), block, 0, st, rowptr, m, cap, rx.totals, w0,
                       rx.starts);
    int last = w1;
    if (rx.passes == 2) {
        hipLaunchKernelGGL((k_rx_move<true, false>), grid, block, 0, st, csr, (int)n, cap, w0,
                           rx.hist, rx.totals, rx.row, rx.val, rx.key);
        hipLaunchKernelGGL(k_rx_count<unsigned long long>, grid, block, 0, st, rowptr, m, cap,
                           rx.key, rx.starts, w0, w1, n, rx.hist, columns);
    } else {
        const int64_t cells = (int64_t)1 << (w0 + w1);
        hipLaunchKernelGGL((k_rx_move<true, false>), grid, block, 0, st, csr, (int)n, cap, w0,
                           rx.hist, rx.totals, rowidx, vals_t, rx.key2);
        hipLaunchKernelGGL(k_tr_zero, dim3(256), dim3(256), 0, st, rowptr, m, (int64_t)-1,
                           rx.counts, cells);
        hipLaunchKernelGGL(k_rx_count<int>, grid, block, 0, st, rowptr, m, cap, rx.key2, rx.starts,
                           w0, w1, cells, rx.hist, rx.counts);
        hipLaunchKernelGGL(k_rx_offsets, digits, block, 0, st, rowptr, m, cap, rx.hist, rx.totals,
                           nullptr, 0);
        hipLaunchKernelGGL(k_rx_starts, dim3(1), block, 0, st, rowptr, m, cap, rx.counts, w0 + w1,
                           rx.starts);
        hipLaunchKernelGGL((k_rx_move<false, false>), grid, block, 0, st, out, (int)n, cap, w1,
                           rx.hist, rx.totals, rx.row, rx.val, rx.key);
        hipLaunchKernelGGL(k_rx_count<unsigned long long>, grid, block, 0, st, rowptr, m, cap,
                           rx.key, rx.starts, w0 + w1, w2, n, rx.hist, columns);
        last = w2;
    }
    hipLaunchKernelGGL(k_rx_offsets, digits, block, 0, st, rowptr, m, cap, rx.hist, rx.totals,
                       nullptr, 0);
    hipLaunchKernelGGL((k_rx_move<false, true>), grid, block, 0, st, mid, (int)n, cap, last,
                       rx.hist, rx.totals, rowidx, vals_t, nullptr);
}

void profile_free(als_ctx* ctx) {
    if (!ctx->prof_ev) return;
    for (int i = 0; i < 4 * ctx->prof_cap; ++i) (void)hipEventDestroy(ctx->prof_ev[i]);
    delete[] ctx->prof_ev;
    ctx->prof_ev = nullptr;
    ctx->prof_cap = ctx->prof_count = 0;
}

}  // namespace

extern "C" {

size_t als_workspace_bytes(int device, int32_t f_max) {
    if (f_max < 1 || f_max > ALS_F_MAX) return 0;
    int cus = 0, w_cap = 0, waves[kMaxNB + 1][kLastForms] = {{0}};
    if (query_device(device, f_max, &cus, waves, &w_cap) != ALS_OK) return 0;
    return make_layout(waves, nb_of(f_max), cus).total;
}

int als_init(als_ctx** out, int device, void* workspace, size_t workspace_bytes, int32_t f_max) {
    if (!out) return ALS_ERR_INVALID_ARG;
    *out = nullptr;
    if (f_max < 1 || f_max > ALS_F_MAX) return ALS_ERR_UNSUPPORTED_F;
    if (!workspace) return ALS_ERR_WORKSPACE;
    if (!aligned(workspace, 256)) return ALS_ERR_ALIGN;
    als_ctx* ctx = new (std::nothrow) als_ctx();
    if (!ctx) return ALS_ERR_INVALID_ARG;
    int rc = query_device(device, f_max, &ctx->cus, ctx->waves, &ctx->w_cap,
                          &ctx->lds_per_block);
    if (rc != ALS_OK) { delete ctx; return rc; }
    ctx->device = device;
    ctx->f_max = f_max;
    {
        const char* g = getenv("ALS_GATHER");
        ctx->global_gather = g && strcmp(g, "global") == 0;
        ctx->staged_gather = g && strcmp(g, "lds") == 0;
        const char* t = getenv("ALS_LAST_BLOCK");
        ctx->tile_last_block = t && strcmp(t, "tiles") == 0;
        // part length in entries: kPart, or ALS_PART_ENTRIES rounded down to a power of two
        // times the entries of a pipeline group (at least one group)
        int64_t part = kPart;
        const char* pe = getenv("ALS_PART_ENTRIES");
        if (pe && atoll(pe) > 0) part = atoll(pe);
        int groups = 1;
        while ((int64_t)kGroupEntries * groups * 2 <= part && groups < (1 << 24)) groups *= 2;
        ctx->part_groups = groups;
    }
    ctx->nb_max = nb_of(f_max);
    if (int su = noalloc_setup(device); su != ALS_OK) { delete ctx; return su; }
    if (ctx->staged_gather) {   // the staged form's residency bounds the partition's W
        DeviceGuard g2(device);
        for (int nb = 1; nb <= ctx->nb_max; ++nb) {
            int w = 0;
            if (staged_waves_for_nb(nb, ctx->cus, &w) != 0) { delete ctx; return ALS_ERR_HIP; }
            if (w < ctx->waves[nb][kLastTiles]) ctx->waves[nb][kLastTiles] = w;
        }
    }
    ctx->lay = make_layout(ctx->waves, ctx->nb_max, ctx->cus);
    if (workspace_bytes < ctx->lay.total) { delete ctx; return ALS_ERR_WORKSPACE; }
    ctx->ws = (unsigned char*)workspace;
    ctx->ws_bytes = workspace_bytes;
    DeviceGuard guard(device);
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, nullptr,
                       (unsigned long long*)(ctx->ws + ctx->lay.status));
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) { delete ctx; return ALS_ERR_HIP; }
    *out = ctx;
    return ALS_OK;
}

int als_destroy(als_ctx* ctx) {
    if (ctx) {
        DeviceGuard guard(ctx->device);
        profile_free(ctx);
    }
    delete ctx;
    return ALS_OK;
}

int als_profile_begin(als_ctx* ctx, int32_t capacity) {
    if (!ctx || capacity < 1) return ALS_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    profile_free(ctx);
    ctx->prof_ev = new (std::nothrow) hipEvent_t[4 * (size_t)capacity];
    if (!ctx->prof_ev) return ALS_ERR_INVALID_ARG;
    for (int i = 0; i < 4 * capacity; ++i) {
        hipError_t e = hipEventCreate(&ctx->prof_ev[i]);
        if (e != hipSuccess) {
            for (int j = 0; j < i; ++j) (void)hipEventDestroy(ctx->prof_ev[j]);
            delete[] ctx->prof_ev;
            ctx->prof_ev = nullptr;
            return fail_hip(ctx, e);
        }
    }
    ctx->prof_cap = capacity;
    ctx->prof_count = 0;
    return ALS_OK;
}

int als_profile_end(als_ctx* ctx, float* ms_out, int32_t capacity, int32_t* count_out) {
    if (!ctx || !count_out || (capacity > 0 && !ms_out)) return ALS_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    *count_out = 0;
    if (!ctx->prof_ev) return ALS_OK;
    const int cnt = ctx->prof_count < capacity ? ctx->prof_count : capacity;
    int rc = ALS_OK;
    if (ctx->prof_count > 0) {
        hipError_t e = hipEventSynchronize(ctx->prof_ev[4 * (ctx->prof_count - 1) + 3]);
        if (e != hipSuccess) rc = fail_hip(ctx, e);
    }
    for (int i = 0; i < cnt && rc == ALS_OK; ++i)
        for (int k = 0; k < 3; ++k) {
            float ms = 0.f;
            hipError_t e = hipEventElapsedTime(&ms, ctx->prof_ev[4 * i + k], ctx->prof_ev[4 * i + k + 1]);
            if (e != hipSuccess) { rc = fail_hip(ctx, e); break; }
            ms_out[3 * i + k] = ms;
        }
    *count_out = cnt;
    profile_free(ctx);
    return rc;
}

int als_half_sweep(als_ctx* ctx, const int64_t* rowptr, const int32_t* colidx, const float* vals,
                   int64_t m, int64_t n, int32_t f, float lambda, const float* theta_in,
                   float* x_out, void* stream) {
    if (!ctx) return ALS_ERR_INVALID_ARG;
    if (f < 1 || f > ctx->f_max) return ALS_ERR_UNSUPPORTED_F;
    if (m < 0 || n < 0 || !(lambda >= 0.f) || !std::isfinite(lambda)) return ALS_ERR_INVALID_ARG;
    if (m == 0) return ALS_OK;
    if (!rowptr || !x_out || (n > 0 && (!colidx || !vals || !theta_in))) return ALS_ERR_INVALID_ARG;
    if (!aligned(rowptr, 8) || !aligned(colidx, 4) || !aligned(vals, 4) ||
        !aligned(theta_in, 4) || !aligned(x_out, 4))
        return ALS_ERR_ALIGN;
    if (theta_in && n > 0) {
        const char* t0 = (const char*)theta_in;
        const char* t1 = t0 + sizeof(float) * (size_t)n * (size_t)f;
        const char* x0 = (const char*)x_out;
        const char* x1 = x0 + sizeof(float) * (size_t)m * (size_t)f;
        if (t0 < x1 && x0 < t1) return ALS_ERR_ALIAS;
    }
    if (ctx->staged_gather && !staged_supported(n, f)) return ALS_ERR_UNSUPPORTED_F;
    const int nb = nb_of(f);
    const int W = ctx->waves[nb][form_of(ctx, f)];
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipStream_t st = (hipStream_t)stream;
    switch (nb) {
        case 1: launch_sweep<1>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 2: launch_sweep<2>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 3: launch_sweep<3>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 4: launch_sweep<4>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 5: launch_sweep<5>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 6: launch_sweep<6>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 7: launch_sweep<7>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 8: launch_sweep<8>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        case 9: launch_sweep<9>(ctx, rowptr, colidx, vals, m, n, f, lambda, theta_in, x_out, st, W); break;
        default: return ALS_ERR_UNSUPPORTED_F;
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ALS_OK : fail_hip(ctx, e);
}

int als_rmse(als_ctx* ctx, const int64_t* rowptr, const int32_t* colidx, const float* vals,
             int64_t m, int64_t n, int32_t f, const float* x, const float* theta,
             double* rmse_out, void* stream) {
    if (!ctx) return ALS_ERR_INVALID_ARG;
    const int rc = rmse_check(rowptr, colidx, vals, m, n, f, x, theta, rmse_out);
    if (rc != ALS_OK) return rc;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipError_t e = rmse_launch(ctx->cus, 4 * ctx->rmse_waves_per_simd, ctx->global_gather,
                               (hipStream_t)stream, rowptr, colidx, vals, m, n, f, x, theta,
                               (double*)(ctx->ws + ctx->lay.rmse),
                               (unsigned*)(ctx->ws + ctx->lay.status + 128), rmse_out);
    return e == hipSuccess ? ALS_OK : fail_hip(ctx, e);
}

int als_rmse_noalloc(int device, const int64_t* rowptr, const int32_t* colidx,
                     const float* vals, int64_t m, int64_t n, int32_t f, const float* x,
                     const float* theta, double* rmse_out, void* stream) {
    const int rc = rmse_check(rowptr, colidx, vals, m, n, f, x, theta, rmse_out);
    if (rc != ALS_OK) return rc;
    const int su = noalloc_setup(device);
    if (su != ALS_OK) return su;
    const NoAllocDevice& d = g_noalloc[device];
    // the partials of the device's fixed chunk count must fit the fixed array
    if (kNoAllocPartials + sizeof(double) * (size_t)d.cus * kRmseWavesPerCU > kNoAllocScratchBytes)
        return ALS_ERR_WORKSPACE;
    DeviceGuard guard(device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipError_t e = rmse_launch(d.cus, 0, false, (hipStream_t)stream, rowptr, colidx, vals, m, n,
                               f, x, theta, (double*)(d.ptr + kNoAllocPartials),
                               (unsigned*)d.ptr, rmse_out);
    return e == hipSuccess ? ALS_OK : ALS_ERR_HIP;
}

int als_status(als_ctx* ctx, void* stream, int64_t* nonspd_rows) {
    if (!ctx || !nonspd_rows) return ALS_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipStream_t st = (hipStream_t)stream;
    unsigned long long host = 0;
    auto* dev = (unsigned long long*)(ctx->ws + ctx->lay.status);
    hipError_t e = hipMemcpyAsync(&host, dev, sizeof host, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return fail_hip(ctx, e);
    hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, st, dev);
    e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(ctx, e);
    *nonspd_rows = (int64_t)host;
    return ALS_OK;
}

int als_plan(als_ctx* ctx, const int64_t* rowptr, int64_t m, int32_t f, int64_t* bounds_out,
             int64_t capacity, int64_t* params_out, void* stream) {
    if (!ctx || !rowptr || !bounds_out || !params_out || m < 0) return ALS_ERR_INVALID_ARG;
    if (f < 1 || f > ctx->f_max) return ALS_ERR_UNSUPPORTED_F;
    if (!aligned(rowptr, 8) || !aligned(bounds_out, 8)) return ALS_ERR_ALIGN;
    const int W = ctx->waves[nb_of(f)][form_of(ctx, f)];
    const int C = chunks_of(W);
    params_out[0] = C;
    params_out[1] = kCostPerEntry;
    params_out[2] = row_cost(f);
    params_out[3] = kSnap;
    params_out[4] = W;
    params_out[5] = kTailDiv;
    if (capacity < C + 1) return ALS_ERR_INVALID_ARG;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipLaunchKernelGGL(k_plan, dim3((C + 1 + 63) / 64), dim3(64), 0, (hipStream_t)stream, rowptr,
                       m, W, C, (int64_t)kCostPerEntry, row_cost(f), (int64_t)kSnap, bounds_out,
                       nullptr, nullptr);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ALS_OK : fail_hip(ctx, e);
}

int als_csr_to_csc(als_ctx* ctx, const int64_t* rowptr, const int32_t* colidx, const float* vals,
                   int64_t m, int64_t n, int64_t* colptr, int32_t* rowidx, float* vals_t,
                   void* stream) {
    if (!ctx || !rowptr || !colptr || m < 0 || n < 0 || m > INT32_MAX) return ALS_ERR_INVALID_ARG;
    if (m > 0 && n > 0 && (!colidx || !vals || !rowidx || !vals_t)) return ALS_ERR_INVALID_ARG;
    if (!aligned(rowptr, 8) || !aligned(colptr, 8) || !aligned(colidx, 4) || !aligned(vals, 4) ||
        !aligned(rowidx, 4) || !aligned(vals_t, 4))
        return ALS_ERR_ALIGN;
    // scratch: everything past the status block (no half-sweep runs meanwhile on this context)
    const size_t tiles = (size_t)(n + kScanTile - 1) / kScanTile;
    const size_t sums_bytes = align256(sizeof(int64_t) * (tiles + 1));
    const size_t avail = ctx->ws_bytes - ctx->lay.bounds;
    if (avail < sums_bytes + sizeof(int32_t) * (size_t)(n > 0 ? n : 1)) return ALS_ERR_WORKSPACE;
    int64_t R = n > 0 ? (int64_t)((avail - sums_bytes) / (sizeof(int32_t) * (size_t)n)) : 1;
    const int64_t r_cap = (int64_t)ctx->cus * kTransposeWavesPerCU;
    if (R > r_cap) R = r_cap;
    if (R > m) R = m;
    if (R < 1) R = 1;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipStream_t st = (hipStream_t)stream;
    unsigned char* base = ctx->ws + ctx->lay.bounds;
    int64_t* sums = (int64_t*)base;
    int32_t* cnt = (int32_t*)(base + sums_bytes);
    // The sort runs when the entries fit beside its counters, the counting passes otherwise.  The
    // number of entries is known on the device only (m n does not bound it: entries with a column
    // outside [0, n) are among them), so both are launched and the one that does not run returns at
    // once (about 2 us a kernel).
    RxSpace rx;
    const bool any = m > 0 && n > 0;
    const int64_t cap = any ? rx_layout(base + sums_bytes, avail - sums_bytes, n, &rx) : 0;
    const size_t lds_bytes = sizeof(int32_t) * (size_t)(n > 0 ? n : 1);
    const bool lds = n <= kTrLdsCols && lds_bytes <= ctx->lds_per_block;
    if (n > 0) {   // colptr: the columns' counts (of the sort), then their scan
        const int64_t words = 2 * n, zb = (words + 255) / 256;
        hipLaunchKernelGGL(k_tr_zero, dim3((unsigned)(zb < 4096 ? zb : 4096)), dim3(256), 0, st,
                           rowptr, m, (int64_t)-1, (int32_t*)colptr, words);
    }
    if (cap > 0)
        rx_launch(rx, cap, st, rowptr, colidx, vals, m, n, colptr, (uint32_t*)rowidx, vals_t);
    if (any) {
        // LDS counters when one row block's fit in a workgroup's LDS
        if (lds) {
            hipError_t ea = hipFuncSetAttribute((const void*)k_tr_count_lds,
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)lds_bytes);
            if (ea == hipSuccess)
                ea = hipFuncSetAttribute((const void*)k_tr_scatter_lds,
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)lds_bytes);
            if (ea != hipSuccess) return fail_hip(ctx, ea);
        }
        const int64_t cells = R * n, zb = (cells + 255) / 256;
        hipLaunchKernelGGL(k_tr_zero, dim3((unsigned)(zb < 4096 ? zb : 4096)), dim3(256), 0, st,
                           rowptr, m, cap, cnt, cells);
        if (lds)
            hipLaunchKernelGGL(k_tr_count_lds, dim3((unsigned)R), dim3(256), lds_bytes, st, rowptr,
                               colidx, m, (int)n, cap, (int)R, cnt);
        else
            hipLaunchKernelGGL(k_tr_count, dim3((unsigned)R), dim3(256), 0, st, rowptr, colidx,
                               m, n, cap, (int)R, cnt);
        hipLaunchKernelGGL(k_tr_colscan, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                           rowptr, m, n, cap, (int)R, cnt, colptr);
    }
    if (n > 0)
        hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)tiles), dim3(256), 0, st, colptr, n, sums);
    hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, st, sums, (int64_t)tiles, colptr, n);
    if (n > 0)
        hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)tiles), dim3(256), 0, st, colptr, n, sums);
    if (any) {
        if (lds)
            hipLaunchKernelGGL(k_tr_scatter_lds, dim3((unsigned)R), dim3(kWave), lds_bytes, st,
                               rowptr, colidx, vals, m, (int)n, cap, (int)R, cnt, colptr, rowidx,
                               vals_t);
        else
            hipLaunchKernelGGL(k_tr_scatter, dim3((unsigned)R), dim3(kWave), 0, st, rowptr,
                               colidx, vals, m, n, cap, (int)R, cnt, colptr, rowidx, vals_t);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ALS_OK : fail_hip(ctx, e);
}

int als_gather_dump(als_ctx* ctx, const int64_t* rowptr, const int32_t* colidx,
                    const float* vals, int64_t m, int64_t n, int32_t f, const float* theta,
                    int64_t u, float* out, int64_t capacity, void* stream) {
    if (!ctx) return ALS_ERR_INVALID_ARG;
    if (f < 1 || f > ctx->f_max) return ALS_ERR_UNSUPPORTED_F;
    if (m < 1 || n < 0 || u < 0 || u >= m || capacity < 0 || !rowptr || !out)
        return ALS_ERR_INVALID_ARG;
    if (n > 0 && (!colidx || !vals || !theta)) return ALS_ERR_INVALID_ARG;
    if (!aligned(rowptr, 8) || !aligned(colidx, 4) || !aligned(vals, 4) || !aligned(theta, 4) ||
        !aligned(out, 4))
        return ALS_ERR_ALIGN;
    if (ctx->staged_gather && !staged_supported(n, f)) return ALS_ERR_UNSUPPORTED_F;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return ALS_ERR_DEVICE;
    hipStream_t st = (hipStream_t)stream;
    const int nb = nb_of(f);
    const int64_t limit = capacity / (16 * (nb + 3));
    switch (nb) {
#define ALS_DUMP_CASE(NB)                                                                     \
        case NB:                                                                              \
            launch_dump<NB>(ctx, rowptr, colidx, vals, n, f, theta, u, out, limit, st);       \
            break;
        ALS_DUMP_CASE(1) ALS_DUMP_CASE(2) ALS_DUMP_CASE(3) ALS_DUMP_CASE(4) ALS_DUMP_CASE(5)
        ALS_DUMP_CASE(6) ALS_DUMP_CASE(7) ALS_DUMP_CASE(8) ALS_DUMP_CASE(9)
#undef ALS_DUMP_CASE
        default: return ALS_ERR_UNSUPPORTED_F;
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ALS_OK : fail_hip(ctx, e);
}

int als_rmse_waves(als_ctx* ctx, int32_t waves_per_simd) {
    if (!ctx || waves_per_simd < 0 || waves_per_simd > kRmseWavesPerCU / 4)
        return ALS_ERR_INVALID_ARG;
    ctx->rmse_waves_per_simd = waves_per_simd;
    return ALS_OK;
}

int als_last_hip_error(const als_ctx* ctx) { return ctx ? ctx->last_hip : 0; }

const char* als_strerror(int status) {
    switch (status) {
        case ALS_OK: return "ok";
        case ALS_ERR_INVALID_ARG: return "invalid argument";
        case ALS_ERR_UNSUPPORTED_F: return "f outside the supported range";
        case ALS_ERR_WORKSPACE: return "workspace missing or too small";
        case ALS_ERR_ALIGN: return "pointer not naturally aligned";
        case ALS_ERR_HIP: return "HIP runtime error";
        case ALS_ERR_ALIAS: return "theta_in and x_out overlap";
        case ALS_ERR_DEVICE: return "invalid or unsupported device";
        default: return "unknown status";
    }
}

}  // extern "C"
