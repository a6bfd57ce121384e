// fused.hip -- teacher log-probabilities from the output projection, logits never stored.
//
// Eq. (1) (Sec. 3.1) with the teacher's logits z = h W^T, h the teacher's final
// hidden state of the row ([N, d] bf16) and W its lm_head weight as stored by a
// linear layer ([V, d] bf16, row v = the weights of vocabulary entry v):
// log pi_T(y) = z_y - log sum_v exp(z_v).  The [N, V] logits (40 GB at the
// fused workload) exist only tile by tile in registers.
//
// Kernel 1 (MFMA): a 256 x 256 tile of z per workgroup of eight waves, two per
//   SIMD, each wave holding a 128 (vocabulary) x 64 (token) fp32 accumulator
//   (32 v_mfma_f32_16x16x32_bf16 tiles, 128 registers).  The 16 x 16 form reads and
//   writes half as many accumulator registers per product as the 32 x 32 one, and
//   under this load the chip's power, not its issue rate, sets the pace.  The waves
//   form two groups of four (one wave per SIMD) that alternate every 32-wide K step: while one
//   group multiplies from registers, the other reads its next fragments from LDS
//   and issues loads, then a barrier swaps them (ping-pong), so each SIMD's matrix
//   unit always has a wave with work.  K = d streams in 64-wide stages through a
//   ring of five 32 KB LDS buffers (the whole 160 KB LDS), each holding one
//   operand of one stage, filled by direct buffer->LDS loads (buffer_load_dwordx4
//   ... lds, no register staging): W of stage j in buffer 2j mod 5, H in 2j+1 mod 5.
//   Every memory phase issues one operand's loads -- H(j+1) in the first half of
//   stage j, W(j+2) in the second -- so the loads are spread evenly over the
//   phases and each has two to four phases to land.  Eight lanes load one row's
//   128 bytes, a whole cache line, and rows are XOR-swizzled so the 16-byte
//   fragment reads are free of bank conflicts.  No vector ALU work remains in the
//   loop: wave-uniform values are scalar and the fragment addresses are fixed per
//   buffer.  Both operands are K-contiguous, so each MFMA operand is one 16-byte
//   LDS read.  W is the A operand and H the B operand, so each lane's
//   accumulators hold 32 of one token's 128 logits and the lanes l ^ 16, l ^ 32 and
//   l ^ 48 the other 96: the epilogue reduces a token to (max, sum of exp(z - max))
//   with two exchanges and writes it to a partial table [V/128][N] (tokens
//   contiguous).
//   Workgroups are numbered so that the 32 resident on one XCD (dispatch is
//   round-robin over the 8 XCDs) cover a 4 x 8 block of tiles of a 16 x 16
//   super-tile: each XCD's L2 serves every H panel slice to 8 tiles and every
//   W slice to 4.  Super-rows are grouped in bands (up to 128 MiB of H, eight
//   super-rows at d = 2,048) and a band is walked one super-column at a time:
//   the band's H and the current W slab both stay in the 256 MB last-level
//   cache, so each W slab comes from HBM once per band instead of once per
//   super-row.  Row tiles and vocabulary tiles past the last whole super-tile
//   are numbered apart, without holes (tile_of), so that every XCD and every
//   shader engine of it has the same share of them.
//   Up to 128 rows a kernel of its own streams W through registers (fused_rows).
// Kernel 2: z_y = h . w_y per row (one wave per row, fp32), the merge of each row's V/128
//   partials, and log pi_T(y) = (z_y - m) - log s.
#include <atomic>

#include "common.hpp"

namespace stride {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))

constexpr int kBM = 256, kBN = 256, kBK = 64;      // tile and stage width along K
constexpr int kThreads = 512;                      // eight waves
constexpr int kRowB = kBK * 2;                     // 128 bytes per LDS row
constexpr int kBufB = kBM * kRowB;                 // 32 KB: one operand of one stage
constexpr int kBuffers = 5;                        // LDS ring of operand buffers
constexpr size_t kLdsBytes = (size_t)kBuffers * kBufB;  // 160 KB, the whole LDS
constexpr int kHalf = 128;                         // vocabulary entries per partial
// H bytes a band of super-rows may hold in the 256 MB last-level cache beside the W slab
// it is reading: 128 MiB, eight 4,096-row super-rows at d = 2,048
constexpr int64_t kBandHBytes = 128ll << 20;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.69314718055994531f;
// Lowest reference point of a (max, sum): times log2(e) it is still finite in fp32, so logits below it
// add nothing to the row, whether or not the others of their partial are as low.
constexpr float kLowestRef = -2.358e38f;
// Third word of a raw buffer descriptor: 32-bit data format, no swizzle; accesses
// at or beyond num_records bytes return zeros.
constexpr int kBufferFlags = 0x00020000;

struct FusedArgs {
    const uint16_t *h;     // [N, d]
    const uint16_t *w;     // [V, d]
    float2 *partial;       // [n_half, N]
    int64_t n_rows;
    int32_t vocab;
    int32_t d;
    int32_t n_half;
    int32_t tiles_m, tiles_n;
    int32_t super_rows, super_cols;  // whole super-tiles of 16 x 16 tiles along rows and vocabulary
    int64_t blocks;        // workgroups that the tiles are numbered over
    int32_t band;          // super-rows per band; a band is walked one super-column at a time
};

__device__ __forceinline__ float ex2(float x) { return __builtin_amdgcn_exp2f(x); }

// 16-byte chunk c of LDS row r is stored at position c ^ swz(r).  The LDS has 64
// banks (256 B per cycle) and serves a 16-byte-per-lane read in four cycles of 16
// lanes; on gfx950 a cycle takes four lane quads of one half-wave, quads 0, 3, 5, 6
// or quads 1, 2, 4, 7 (the quads whose index has even or odd parity; measured with
// the bank-conflict counter).  Rows are 128 B, so a row's place in the 256-byte bank
// row is r % 2.  Fragment lane l reads row l % 16 (of a 16-row block) at chunk
// 4 * hf + l / 16 for the half hf of the stage; over the 16 lanes of either kind of
// cycle the pairs (r % 2, chunk ^ swz(r)) are all distinct, so every read is free of
// conflicts.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Wait until at most N vector-memory operations of this wave are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmem() {
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

// Wait until this wave's LDS reads have returned.
__device__ __forceinline__ void wait_lds() {
    __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (0 << 8) | (3 << 14));
}

__device__ __forceinline__ void barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

// Tile (row tile tm, vocabulary tile tn) of workgroup b.  Three regions, one after the other:
//   A  whole super-tiles, 256 workgroups each, in bands of super-rows;
//   B  the vocabulary tiles past the last whole super-column, for the rows of region A: each XCD
//      takes an eighth of the row tiles;
//   C  the row tiles past the last whole super-row (up to 15), for every vocabulary tile, in
//      one strip of up to 8 row tiles or two: XCD x takes the vocabulary tiles x, x + 8, ... and
//      all the strip's rows of each in turn.
// Every number in A and B is a tile, and in C all but the last vocabulary tiles' of some XCDs.
// Holes cost more than their own empty workgroups: an XCD hands consecutive workgroups to its
// four shader engines in turn, so numbering a single row tile as the first of a block of four
// left three quarters of the chip idle.  Measured with V = 151,936, d = 2,048: 431 us for 64 to
// 512 rows with such holes, 213 to 280 us without; 5,000 rows 3.56 ms against 2.19 ms.
__host__ __device__ inline int strip_rows(int rem) { return rem > 8 ? (rem + 1) / 2 : rem; }

__device__ __forceinline__ void tile_of(const FusedArgs &a, int b, int &tm, int &tn) {
    const int xcd = b & 7;
    int s = b >> 3;
    const int n_a = a.super_rows * a.super_cols * 32;  // per XCD
    if (s < n_a) {
        const int S = s >> 5, q = s & 31;
        // super-tile S -> (super-row, super-column): bands of a.band super-rows, each band
        // walked column by column, so a W slab read from HBM serves the whole band from the
        // last-level cache while the band's H stays there too
        const int per_band = a.band * a.super_cols;
        const int bi = S / per_band, r0 = bi * a.band, idx = S - bi * per_band;
        const int rows_b = (a.super_rows - r0) < a.band ? (a.super_rows - r0) : a.band;
        tm = (r0 + idx % rows_b) * 16 + (xcd >> 1) * 4 + (q & 3);
        tn = (idx / rows_b) * 16 + (xcd & 1) * 8 + (q >> 2);
        return;
    }
    s -= n_a;
    const int cols = a.tiles_n - a.super_cols * 16, n_b = a.super_rows * 2 * cols;
    if (s < n_b) {
        tm = xcd * a.super_rows * 2 + s / cols;
        tn = a.super_cols * 16 + s % cols;
        return;
    }
    s -= n_b;
    const int per_xcd = (a.tiles_n + 7) >> 3;
    tm = a.super_rows * 16;
    int h = strip_rows(a.tiles_m - tm);
    if (s >= h * per_xcd) {
        s -= h * per_xcd;
        tm += h;
        h = a.tiles_m - tm;
    }
    tm += s % h;
    tn = (s / h) * 8 + xcd;
}

// Fold one partial (max p.x, sum p.y of exp(z - p.x)) into a running (m, s).
__device__ __forceinline__ void fold_partial(float &m, float &s, const float2 p) {
    const float mn = fmaxf(m, p.x);
    const float ref = (mn == -INFINITY) ? 0.0f : mn;
    s = s * ex2((m - ref) * kLog2e) + p.y * ex2((p.x - ref) * kLog2e);
    m = mn;
}

// NB: 16-row vocabulary blocks per wave; the tile holds 32 NB vocabulary entries.
template <bool kAlone, int NB>
__device__ __forceinline__ void fused_lse(const FusedArgs &a) {
    constexpr int kBN = 32 * NB, kWaveV = 16 * NB;  // vocabulary entries of the tile and of a wave
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    // wave-uniform values in scalar registers: the LDS-DMA destinations are scalar arithmetic
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2;                   // ping-pong group (one wave per SIMD)
    const int wv = wave & 1, wt = wave >> 1;     // vocabulary half, token quarter

    // ---- tile of this workgroup (XCD-aware order) ----
    int tm, tn;
    const int64_t b = block_index<kThreads>();
    if (b >= a.blocks) return;
    tile_of(a, (int)b, tm, tn);
    if (tm >= a.tiles_m || tn >= a.tiles_n) return;
    const int64_t m0 = (int64_t)tm * kBM;
    const int64_t n0 = (int64_t)tn * kBN;
    const int d = a.d, ns = d / kBK;
    // kAlone (one row tile, so no other tile shares this one's W): a tile starts at a K stage of its
    // own.  With all of them at the same column of W's rows, the reads crowd on a part of the
    // memory channels (218 rows, d = 2,048: 200 -> 171 us; 200 rows, d = 4,096: 358 -> 289).  Tiles
    // that share W keep the common start, so that they meet its lines in L2, and have no scalar
    // work for it in the loop (which took 1 to 2% of a large call).
    const int rot = kAlone ? tn % ns : 0;

    // ---- direct global -> LDS loads (buffer_load_dwordx4 ... lds): for each operand and
    // stage, each wave fills 32 rows of that operand's buffer, 8 rows per instruction (lane l
    // -> row l >> 3, position l & 7 of the swizzled row).  Each operand's descriptor spans
    // only the rows of this tile that exist, so rows past N or V read as zeros (their results
    // are never used) and no load can leave the operand.  Lane offsets are 32-bit; the K
    // position goes in the scalar offset.
    const int64_t h_rows = (a.n_rows - m0) < kBM ? (a.n_rows - m0) : kBM;
    const int64_t w_rows = (a.vocab - n0) < kBN ? (a.vocab - n0) : kBN;
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.h + m0 * d), (short)0, (int)(h_rows * d * 2), kBufferFlags);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.w + n0 * d), (short)0, (int)(w_rows * d * 2), kBufferFlags);
    const int lr = lane >> 3, lp = lane & 7;
    int voff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int R = 32 * wave + 8 * i + lr;
        voff[i] = (R * d + ((lp ^ swz(R)) * 8)) * 2;
    }
    auto issue = [&](const __amdgpu_buffer_rsrc_t &rsrc, int j, int buf) __attribute__((always_inline)) {
        char *dst = lds + buf * kBufB;
        int k = j;
        if (kAlone) {
            k += rot;
            if (k >= ns) k -= ns;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsrc, LDS_PTR(dst + (32 * wave + 8 * i) * kRowB), 16, voff[i], k * kRowB, 0, 0);
    };

    // ---- MFMA fragments: W is the A operand and H the B operand of 16 x 16 x 32 products,
    // so lane l's accumulators hold token jj*16 + l%16 and 4 vocabulary entries of each
    // 16-row block.  Lane l reads row l % 16 of a block at chunk 4*hf + l/16; the fragment
    // addresses are fixed per buffer pair {0,1}, {2,3}, {4} and stage half: the buffer's
    // place in its pair and the 16-row block go in the read's immediate offset.
    const int fr = lane & 15, kg = lane >> 4;
    int wb[3][2], hb[3][2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const int f = fr * kRowB + (((4 * hf + kg) ^ swz(fr)) * 16);
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            wb[g][hf] = g * 2 * kBufB + (wv * kWaveV) * kRowB + f;
            hb[g][hf] = g * 2 * kBufB + (wt * 64) * kRowB + f;
            // opaque to the compiler: it would otherwise fold the pair's 64 KB step into the
            // reads' offsets, overflow their 16-bit immediate and keep a register per read
            asm volatile("" : "+v"(wb[g][hf]), "+v"(hb[g][hf]));
        }
    }
    bf16x8 FA[NB], FB[4];
    f32x4 acc[NB][4];  // the first K step's MFMAs start from zero, so no vector moves clear it

    // One 32-wide K step of this wave (half hf of stage j, whose H and W operands sit in
    // buffers hbuf and wbuf): fragments from LDS and one operand's loads, then the MFMAs.
    // The two groups are one phase apart, so every barrier is met by all eight waves: group
    // 0 at the end of a memory phase when group 1 ends a compute phase, and the other way
    // round.  The first half-stage loads H(j+1) into the buffer of W(j-1); the second loads
    // W(j+2) into the buffer of H(j-1) (both read for the last time in stage j-1) and waits
    // until this wave's shares of H(j+1) and W(j+1) have landed, so stage j+1 is complete in
    // LDS at the barrier that ends stage j.  W has the longer window: it comes from HBM where
    // few row tiles share it (300 rows 249 -> 240 us, 1,000 rows 468 -> 462, 4,096 rows 1,717 ->
    // 1,708, 16,384 rows the same, against H having it).
    // may_start: this call site can be the tile's first K step (stage 0 sits at ring position 0),
    // whose MFMAs take zero as their accumulator input.
    auto phase = [&](int j, int hf, int hbuf, int wbuf, bool may_start) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NB; ++t)
            FA[t] = *reinterpret_cast<const bf16x8 *>(lds + wb[wbuf >> 1][hf] + (wbuf & 1) * kBufB +
                                                      t * 16 * kRowB);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            FB[t] = *reinterpret_cast<const bf16x8 *>(lds + hb[hbuf >> 1][hf] + (hbuf & 1) * kBufB +
                                                      t * 16 * kRowB);
        if (hf == 0) {
            const int nb = hbuf + 2 >= kBuffers ? hbuf + 2 - kBuffers : hbuf + 2;
            if (j + 1 < ns) issue(rh, j + 1, nb);
        } else {
            const int nb = wbuf + 4 >= kBuffers ? wbuf + 4 - kBuffers : wbuf + 4;
            if (j + 2 < ns) {
                issue(rw, j + 2, nb);
                wait_vmem<4>();
            } else {
                wait_vmem<0>();
            }
        }
        wait_lds();
        barrier();
        if (may_start && j == 0) {
            const f32x4 zero = {};
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(FA[i], FB[jj], zero, 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
                    acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(FA[i], FB[jj], acc[i][jj], 0, 0, 0);
        }
        barrier();
    };
    // W(j) lives in buffer 2j mod 5 and H(j) in buffer 2j+1 mod 5; r = j mod 5 is a
    // compile-time value at every call, so every buffer index is.
    auto stage = [&](int j, int r) __attribute__((always_inline)) {
        const int wbuf = (2 * r) % kBuffers, hbuf = (2 * r + 1) % kBuffers;
        phase(j, 0, hbuf, wbuf, r == 0);
        phase(j, 1, hbuf, wbuf, false);
    };
    // prologue: W(0), H(0), W(1) in flight, W(0) and H(0) landed
    issue(rw, 0, 0);
    issue(rh, 0, 1);
    if (ns > 1) {
        issue(rw, 1, 2);
        wait_vmem<4>();
    } else {
        wait_vmem<0>();
    }
    barrier();
    if (grp == 1) barrier();  // group 1 runs one phase behind
    int j = 0;
    for (; j + 4 < ns; j += 5) {
        stage(j, 0);
        stage(j + 1, 1);
        stage(j + 2, 2);
        stage(j + 3, 3);
        stage(j + 4, 4);
    }
    if (j < ns) stage(j, 0);  // j is a multiple of 5 here
    if (j + 1 < ns) stage(j + 1, 1);
    if (j + 2 < ns) stage(j + 2, 2);
    if (j + 3 < ns) stage(j + 3, 3);
    if (grp == 0) barrier();  // both groups meet the same number of barriers

    // ---- epilogue: per token of this wave, (max, sum exp(z - max)) over its kWaveV entries;
    // lane l holds entries i*16 + 4*(l/16) + e of token jj*16 + l%16, and the lanes l, l^16,
    // l^32, l^48 that share a token combine theirs with two exchanges ----
    const int q4 = lane >> 4;
    const int64_t v_base = n0 + wv * kWaveV;
    const int vlim = (int)((a.vocab - v_base) < kWaveV ? (a.vocab - v_base) : kWaveV);  // valid entries
    const int hidx = tn * 2 + wv;
    float2 both[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        if (vlim < kWaveV) {
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i * 16 + q4 * 4 + e >= vlim) acc[i][jj][e] = -INFINITY;
        }
        float m = acc[0][jj][0];
#pragma unroll
        for (int x = 1; x < 4 * NB; ++x) m = fmaxf(m, acc[x >> 2][jj][x & 3]);
        m = fmaxf(m, __shfl_xor(m, 16, 64));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        const float mref = fmaxf(m, kLowestRef) * kLog2e;
        float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
        for (int x = 0; x < 4 * NB; x += 2) {
            s0 += ex2(__builtin_fmaf(acc[x >> 2][jj][x & 3], kLog2e, -mref));
            s1 += ex2(__builtin_fmaf(acc[(x + 1) >> 2][jj][(x + 1) & 3], kLog2e, -mref));
        }
        float sum = s0 + s1;
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        const int64_t row = m0 + wt * 64 + jj * 16 + (lane & 15);
        if (kAlone) {
            both[jj] = make_float2(m, sum);
        } else if (q4 == 0 && hidx < a.n_half && row < a.n_rows) {
            a.partial[(int64_t)hidx * a.n_rows + row] = make_float2(m, sum);
        }
    }
    if (kAlone) {  // one partial per tile: the second vocabulary half's through LDS
        float2 *half = reinterpret_cast<float2 *>(lds);
        __syncthreads();  // every wave is done with the ring
        if (wv == 1 && q4 == 0) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) half[wt * 64 + jj * 16 + (lane & 15)] = both[jj];
        }
        __syncthreads();
        if (wv == 0 && q4 == 0) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int i = wt * 64 + jj * 16 + (lane & 15);
                fold_partial(both[jj].x, both[jj].y, half[i]);
                if (m0 + i < a.n_rows) a.partial[(int64_t)tn * a.n_rows + m0 + i] = both[jj];
            }
        }
    }
}

__global__ __launch_bounds__(kThreads, 1) void fused_lse_kernel(FusedArgs a) { fused_lse<false, 8>(a); }
__global__ __launch_bounds__(kThreads, 1) void fused_row8_kernel(FusedArgs a) { fused_lse<true, 8>(a); }
__global__ __launch_bounds__(kThreads, 1) void fused_row7_kernel(FusedArgs a) { fused_lse<true, 7>(a); }
__global__ __launch_bounds__(kThreads, 1) void fused_row6_kernel(FusedArgs a) { fused_lse<true, 6>(a); }
__global__ __launch_bounds__(kThreads, 1) void fused_row4_kernel(FusedArgs a) { fused_lse<true, 4>(a); }

// ---- up to 128 rows ----
// The same product where reading W once bounds it (N <= 128): one workgroup per
// CU takes an equal share of the vocabulary for all BT tokens, and streams it without a pause.
// Eight waves of 32 vocabulary entries x BT tokens each; W goes from memory straight into
// registers as MFMA A operands, since no two waves share a row of it, and H through a ring of
// kRing LDS buffers of one 64-wide K stage.  The loads of stage t + 3 are issued when stage t
// begins, so W has three stages to arrive (the tile kernel's window is one and a half, short of
// HBM's latency), and the stages run on across the passes over a workgroup's share.  At the end of a
// pass, though, a wave reads its running (max, sum) from LDS, and such a read waits for all loads into LDS
// that are in flight, so all but the newest stage's W lands first, once for each of the three passes at
// V = 151,936.  A workgroup's K stages start at its own place, so that the chip's W reads, all
// rows at the same column otherwise, spread over the memory channels.  Per token a wave keeps its
// (max, sum) over its passes in LDS; the workgroup writes one partial per token.
constexpr int kRing = 4;
constexpr int kRowsWaves = 8;
constexpr int kShareRows = 32;   // vocabulary entries of a wave and pass
constexpr int kCUs = 256;
// Tokens up to which this kernel takes the call.  Measured against the tile kernel (teacher call,
// V = 151,936, d = 2,048): 16 rows 193 -> 120 us, 64 rows 192 -> 122, 128 rows 192 -> 136.  With
// BT = 256 a wave's 32 entries give two products for each fragment read from LDS and the reads
// bound it: 218 rows 183 us against 174 as one tile row.
constexpr int kMaxRowsN = 128;

template <int BT>
__device__ __forceinline__ void fused_rows(const FusedArgs &a) {
    constexpr int kStage = BT * kRowB;      // H bytes of one stage
    constexpr int kTiles = BT / 16;         // token tiles
    constexpr int kHLoads = BT / 64;        // H loads per wave and stage, 8 rows each
    constexpr int kLoads = kHLoads + 4;     // and all of its loads
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    float2 *part = reinterpret_cast<float2 *>(lds + kRing * kStage) + wave * BT;
    for (int i = lane; i < BT; i += kWave) part[i] = make_float2(-INFINITY, 0.0f);

    // ---- this workgroup's blocks of 32 vocabulary entries, in passes of `per` <= 8 ----
    const int nblk = (a.vocab + kShareRows - 1) / kShareRows;
    const int b0 = (int)((int64_t)nblk * blockIdx.x / gridDim.x);
    const int cnt = (int)((int64_t)nblk * (blockIdx.x + 1) / gridDim.x) - b0;
    const int passes = (cnt + kRowsWaves - 1) / kRowsWaves;
    const int per = (cnt + passes - 1) / passes;
    const int d = a.d, ns = d / kBK, total = passes * ns;
    const int rot = (int)(blockIdx.x % (unsigned)ns);
    const int64_t v0 = (int64_t)b0 * kShareRows;
    const int64_t w_rows = (a.vocab - v0) < (int64_t)cnt * kShareRows ? (a.vocab - v0)
                                                                      : (int64_t)cnt * kShareRows;
    const __amdgpu_buffer_rsrc_t rh = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.h, (short)0, (int)(a.n_rows * d * 2), kBufferFlags);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(a.w + v0 * d), (short)0, (int)(w_rows * d * 2), kBufferFlags);

    int hoff[kHLoads];
#pragma unroll
    for (int i = 0; i < kHLoads; ++i) {
        const int R = (wave * kHLoads + i) * 8 + (lane >> 3);
        hoff[i] = (R * d + (((lane & 7) ^ swz(R)) * 8)) * 2;
    }
    const int fr = lane & 15, kg = lane >> 4;
    const int woff = (fr * d + kg * 8) * 2;  // of the wave's first row; other half + 64 bytes
    u32x4 wreg[kRing][2][2];                 // [stage][16-row block][stage half]
    int ij = 0, iq = 0;                      // stage and pass of the next loads
    auto issue = [&](int slot) __attribute__((always_inline)) {
        int k = ij + rot;
        if (k >= ns) k -= ns;
        char *dst = lds + slot * kStage + wave * kHLoads * 8 * kRowB;
#pragma unroll
        for (int i = 0; i < kHLoads; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rh, LDS_PTR(dst + i * 8 * kRowB), 16, hoff[i],
                                                     k * kRowB, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // the waits below count on H's loads ahead of W's
        // blocks past the share lie past the descriptor: zeros, and no memory traffic
        const int blk = iq * per + wave;
        const int base = wave < per && blk < cnt ? blk * kShareRows * d * 2 : 0x7f000000;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
                wreg[slot][mb][hf] = __builtin_amdgcn_raw_buffer_load_b128(
                    rw, base + woff + mb * 16 * d * 2 + hf * 64, k * kRowB, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (++ij == ns) {
            ij = 0;
            ++iq;
        }
    };
    int hb[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) hb[hf] = fr * kRowB + (((4 * hf + kg) ^ swz(fr)) * 16);

    f32x4 acc[2][kTiles];
    int j = 0, q = 0;  // stage and pass being multiplied
    auto step = [&](int slot) __attribute__((always_inline)) {
        issue((slot + kRing - 1) % kRing);
        const int blk = q * per + wave;
        const bool busy = wave < per && blk < cnt;
        if (busy) {
            if (j == 0) {
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                    for (int jj = 0; jj < kTiles; ++jj) acc[mb][jj] = f32x4{};
            }
            // token fragments in groups of four, the next group's reads ahead of this one's products
            constexpr int kGroups = 2 * kTiles / 4;
            bf16x8 fb[2][4];
            auto read = [&](int g) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int hf = g / (kTiles / 4), jj = g % (kTiles / 4) * 4 + i;
                    fb[g & 1][i] = *reinterpret_cast<const bf16x8 *>(lds + slot * kStage + hb[hf] +
                                                                     jj * 16 * kRowB);
                }
            };
            read(0);
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                const int hf = g / (kTiles / 4);
                if (g + 1 < kGroups) read(g + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb) {
                        const int jj = g % (kTiles / 4) * 4 + i;
                        acc[mb][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, wreg[slot][mb][hf]), fb[g & 1][i], acc[mb][jj], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (++j == ns) {
            j = 0;
            ++q;
            if (busy) {
                // entries mb*16 + 4*kg + e of token jj*16 + fr, as in the tile kernel's epilogue
                const int vlim = (int)(a.vocab - (v0 + (int64_t)blk * kShareRows));
#pragma unroll
                for (int jj = 0; jj < kTiles; ++jj) {
                    float z[8];
#pragma unroll
                    for (int x = 0; x < 8; ++x) {
                        z[x] = acc[x >> 2][jj][x & 3];
                        if (vlim < kShareRows && (x >> 2) * 16 + kg * 4 + (x & 3) >= vlim) z[x] = -INFINITY;
                    }
                    float m = z[0];
#pragma unroll
                    for (int x = 1; x < 8; ++x) m = fmaxf(m, z[x]);
                    m = fmaxf(m, __shfl_xor(m, 16, 64));
                    m = fmaxf(m, __shfl_xor(m, 32, 64));
                    const float mref = fmaxf(m, kLowestRef) * kLog2e;
                    float sum = 0.0f;
#pragma unroll
                    for (int x = 0; x < 8; ++x) sum += ex2(__builtin_fmaf(z[x], kLog2e, -mref));
                    sum += __shfl_xor(sum, 16, 64);
                    sum += __shfl_xor(sum, 32, 64);
                    if (kg == 0) {
                        float2 o = part[jj * 16 + fr];
                        fold_partial(o.x, o.y, make_float2(m, sum));
                        part[jj * 16 + fr] = o;
                    }
                }
            }
        }
        // this wave's H loads of stage t + 1 have landed (W's four of it were issued behind them);
        // after the barrier so have all waves', and this stage's buffer is free
        wait_vmem<2 * kLoads + 4>();
        barrier();
    };
#pragma unroll
    for (int t = 0; t < kRing - 1; ++t) issue(t);
    wait_vmem<2 * kLoads + 4>();
    barrier();
    // Stages past the last pass load h again and no W, and multiply nothing: every load is issued
    // on every path, so the waits count the same loads everywhere.
    for (int t = 0; t < total; t += kRing) {
        step(0);
        step(1);
        step(2);
        step(3);
    }
    wait_vmem<0>();
    __syncthreads();
    const float2 *all = reinterpret_cast<const float2 *>(lds + kRing * kStage);
    for (int i = tid; i < BT; i += kRowsWaves * kWave) {
        float2 o = all[i];
#pragma unroll
        for (int w = 1; w < kRowsWaves; ++w) fold_partial(o.x, o.y, all[w * BT + i]);
        if (i < a.n_rows) a.partial[(int64_t)blockIdx.x * a.n_rows + i] = o;
    }
}

__global__ __launch_bounds__(kRowsWaves *kWave, 1) void fused_rows64_kernel(FusedArgs a) { fused_rows<64>(a); }
__global__ __launch_bounds__(kRowsWaves *kWave, 1) void fused_rows128_kernel(FusedArgs a) { fused_rows<128>(a); }

constexpr int kMergeThreads = 1024;  // 16 waves per workgroup
// Rows from which a merge workgroup takes 64 rows instead of 16: measured, 16 rows take 30.1 us
// against 33.0 at 8,192 rows and 52.0 against 46.8 at 16,384, where every CU has its workgroups
// either way and the longer runs of consecutive rows count.
constexpr int64_t kMergeWide = 12288;

// z_y = h . w_y and the merge of the row's V/128 partials, RW rows per workgroup.  Wave v takes
// the dot products of rows v, v + 16, ... (fp32, one row at a time over all its lanes).  Thread
// (sp, r) folds partials sp, sp + 1024/RW, ... of row r, eight loads in flight, each load
// instruction reading runs of RW consecutive rows (8 RW contiguous bytes); the threads of a row
// are combined by lane exchanges and then through LDS, always in the same order, so the result
// does not depend on timing.
// Latency bounds it while the workgroups are few: at RW = 16 a thread's chain is 1,187 / 64
// folds.  Measured (V = 151,936, d = 2,048) against a merge of four waves per 64 rows (chains
// of 1,187 / 4) after a kernel of its own for z_y: 64 rows 29.3 -> 9.8 us, 4,096 rows 35.7 ->
// 14.7, 16,384 rows 55.5 -> 46.8, 65,536 rows 193 -> 186.
template <int RW>
__global__ __launch_bounds__(kMergeThreads) void fused_merge_kernel(
    const float2 *__restrict__ partial, const uint16_t *__restrict__ h,
    const uint16_t *__restrict__ w, const int32_t *__restrict__ ids, float *__restrict__ logp_t,
    int64_t n_rows, int32_t n_half, int32_t vocab, int32_t d, uint32_t *flags) {
    constexpr int kWaves = kMergeThreads / kWave, kSplit = kMergeThreads / RW;
    __shared__ float2 red[kWaves][RW];
    __shared__ float s_zy[RW];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int r = threadIdx.x & (RW - 1), sp = threadIdx.x / RW;
    const int64_t row0 = block_index<kMergeThreads>() * RW, row = row0 + r;
#pragma unroll
    for (int q = wave; q < RW; q += kWaves) {
        if (row0 + q >= n_rows) break;
        const int32_t y = ids[row0 + q];
        float acc = __builtin_nanf("");
        if (y >= 0 && y < vocab) {
            acc = 0.0f;
            const u32x4 *hp = reinterpret_cast<const u32x4 *>(h + (row0 + q) * d);
            const u32x4 *wp = reinterpret_cast<const u32x4 *>(w + (int64_t)y * d);
            for (int c = lane; c < d / 8; c += kWave) {
                const u32x4 x = hp[c], z = wp[c];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc = __builtin_fmaf(__uint_as_float(x[e] << 16), __uint_as_float(z[e] << 16), acc);
                    acc = __builtin_fmaf(__uint_as_float(x[e] & 0xFFFF0000u),
                                         __uint_as_float(z[e] & 0xFFFF0000u), acc);
                }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, kWave);
        }
        if (lane == 0) s_zy[q] = acc;
    }
    float m = -INFINITY, s = 0.0f;
    if (row < n_rows) {
        const float2 *col = partial + row;
        int j = sp;
        constexpr int U = 8;
        for (; j + (U - 1) * kSplit < n_half; j += U * kSplit) {
            float2 p[U];
#pragma unroll
            for (int u = 0; u < U; ++u) p[u] = col[(int64_t)(j + u * kSplit) * n_rows];
#pragma unroll
            for (int u = 0; u < U; ++u) fold_partial(m, s, p[u]);
        }
        float2 p[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            p[u] = j + u * kSplit < n_half ? col[(int64_t)(j + u * kSplit) * n_rows]
                                           : make_float2(-INFINITY, 0.0f);
#pragma unroll
        for (int u = 0; u < U; ++u) fold_partial(m, s, p[u]);
    }
#pragma unroll
    for (int off = RW; off < kWave; off <<= 1) {
        const float m2 = __shfl_xor(m, off, kWave), s2 = __shfl_xor(s, off, kWave);
        fold_partial(m, s, make_float2(m2, s2));
    }
    if (lane < RW) red[wave][lane] = make_float2(m, s);
    __syncthreads();
    if (threadIdx.x >= RW || row >= n_rows) return;
#pragma unroll
    for (int k = 1; k < kWaves; ++k) fold_partial(m, s, red[k][r]);
    const int32_t y = ids[row];
    uint32_t bad = 0;
    if (!((m > -INFINITY) && (m < INFINITY) && (s > 0.0f) && (s < INFINITY))) bad |= STRIDE_FLAG_NONFINITE;
    if (y < 0 || y >= vocab) bad |= STRIDE_FLAG_TOKEN_OOB;
    const float z = s_zy[r];
    if (!bad && !(z > -INFINITY && z < INFINITY)) bad |= STRIDE_FLAG_NONFINITE;
    if (bad) {
        raise_flag(flags, bad);
        logp_t[row] = __builtin_nanf("");
    } else {
        // z_y comes from its own fp32 dot product and (m, s) from the MFMA accumulators, so
        // their rounding differs by ~1e-6 relative; a log-probability is at most 0, and
        // clamping there only moves a rounding excess toward the true value.
        logp_t[row] = fminf(0.0f, (z - m) - __builtin_amdgcn_logf(s) * kLn2);
    }
}

}  // namespace

namespace {

#ifdef STRIDE_FUSED_BAND_HOOK
std::atomic<int32_t> g_band_override{0};  // super-rows per band; 0: the library's choice
#endif

// The projection kernel's dynamic LDS (160 KB) is above the default limit; the limit is
// raised once per device, so later calls (and calls under stream capture) make no
// attribute call.
hipError_t ensure_lds_limit() {
    static std::atomic<uint64_t> done{0};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (dev >= 0 && dev < 64) ? (1ull << dev) : 0;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    for (const void *f : {reinterpret_cast<const void *>(fused_lse_kernel),
                          reinterpret_cast<const void *>(fused_row8_kernel),
                          reinterpret_cast<const void *>(fused_row7_kernel),
                          reinterpret_cast<const void *>(fused_row6_kernel),
                          reinterpret_cast<const void *>(fused_row4_kernel),
                          reinterpret_cast<const void *>(fused_rows64_kernel),
                          reinterpret_cast<const void *>(fused_rows128_kernel)}) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
        if (e != hipSuccess) return e;
    }
    if (e == hipSuccess && bit) done.fetch_or(bit, std::memory_order_release);
    return e;
}

}  // namespace

namespace {

hipError_t launch_rows(const FusedArgs &a, hipStream_t stream) {
    const int bt = a.n_rows <= 64 ? 64 : 128;
    const size_t lds = (size_t)kRing * bt * kRowB + (size_t)kRowsWaves * bt * sizeof(float2);
    hipLaunchKernelGGL(bt == 64 ? fused_rows64_kernel : fused_rows128_kernel, dim3((unsigned)a.n_half),
                       dim3(kRowsWaves * kWave), lds, stream, a);
    return hipGetLastError();
}

hipError_t launch_merge(const FusedArgs &a, const int32_t *ids, float *logp_t, uint32_t *flags,
                        hipStream_t stream) {
    const int rw = a.n_rows < kMergeWide ? 16 : 64;
    hipLaunchKernelGGL(a.n_rows < kMergeWide ? fused_merge_kernel<16> : fused_merge_kernel<64>,
                       grid_of((a.n_rows + rw - 1) / rw, kMergeThreads), dim3(kMergeThreads), 0, stream,
                       a.partial, a.h, a.w, ids, logp_t, a.n_rows, a.n_half, a.vocab, a.d, flags);
    return hipGetLastError();
}

}  // namespace

size_t fused_ws_bytes(int64_t n_rows, int32_t vocab) {
    const int64_t n_half = ((int64_t)vocab + kHalf - 1) / kHalf;
    // the partial table; the floats after it are spare (the size stays what callers were given)
    return (size_t)n_half * n_rows * sizeof(float2) + (size_t)n_rows * sizeof(float) + 256;
}

hipError_t launch_fused_teacher(const uint16_t *h, const uint16_t *w, const int32_t *ids,
                                float *logp_t, int64_t n_rows, int32_t vocab, int32_t d,
                                uint32_t *flags, void *ws, hipStream_t stream) {
    if (n_rows == 0) return hipSuccess;
    FusedArgs a;
    a.h = h;
    a.w = w;
    a.n_rows = n_rows;
    a.vocab = vocab;
    a.d = d;
    a.n_half = (vocab + kHalf - 1) / kHalf;
    a.tiles_m = (int)((n_rows + kBM - 1) / kBM);
    a.tiles_n = (vocab + kBN - 1) / kBN;
    a.super_rows = a.tiles_m / 16;
    a.super_cols = a.tiles_n / 16;
    const int64_t h_super_row = (int64_t)16 * kBM * d * 2;  // H bytes of one super-row
    int64_t band = kBandHBytes / h_super_row;
#ifdef STRIDE_FUSED_BAND_HOOK
    if (const int32_t o = g_band_override.load()) band = o;
#endif
    if (band > a.super_rows) band = a.super_rows;
    a.band = (int)(band < 1 ? 1 : band);
    a.partial = static_cast<float2 *>(ws);
    hipError_t e = ensure_lds_limit();
    if (e != hipSuccess) return e;
    if (n_rows <= kMaxRowsN) {
        // no more workgroups than partials that the workspace holds; a share's bytes fit the 32-bit
        // range of one descriptor (W of 545 GB and more, host memory that the GPU reads, goes to the tiles)
        const int grid = a.n_half < kCUs ? a.n_half : kCUs;
        if (((int64_t)vocab / grid + 2 * kShareRows) * d * 2 < 0x7f000000) {
            a.n_half = grid;
            e = launch_rows(a, stream);
            if (e != hipSuccess) return e;
            return launch_merge(a, ids, logp_t, flags, stream);
        }
    }
    if (a.tiles_m == 1) {
        // One row tile: of the tile heights built (32 n entries), the one that takes least.  A round
        // of tiles over the 256 CUs took time like n + 6 (d = 2,048; three rounds of n = 8 154 us, three
        // of 7 143, four of 6 168, five of 4 186).  Measured, n = 8 -> the one chosen: 218 rows,
        // V = 151,936 172 -> 161 us (n = 7); 200 rows, V = 81,000 104 -> 89 (6), 50,000 56 -> 53 (7),
        // d = 4,096, V = 20,000 81 -> 62 (4).
        int nb = 8;
        int64_t least = INT64_MAX;
        for (const int n : {8, 7, 6, 4}) {
            const int64_t tiles = ((int64_t)vocab + 32 * n - 1) / (32 * n);
            const int64_t cost = (tiles + kCUs - 1) / kCUs * (n + 6);
            if (cost < least) {
                least = cost;
                nb = n;
            }
        }
        a.tiles_n = (vocab + 32 * nb - 1) / (32 * nb);
        a.super_cols = a.tiles_n / 16;
        a.n_half = a.tiles_n;  // one partial per tile, at most one per 128 entries
        a.blocks = 8 * ((a.tiles_n + 7) / 8);
        hipLaunchKernelGGL(nb == 8 ? fused_row8_kernel : (nb == 7 ? fused_row7_kernel
                                                                 : (nb == 6 ? fused_row6_kernel : fused_row4_kernel)),
                           grid_of(a.blocks, kThreads), dim3(kThreads), kLdsBytes, stream, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_merge(a, ids, logp_t, flags, stream);
    }
    const int64_t rem = a.tiles_m - a.super_rows * 16;
    a.blocks = 8 * ((int64_t)a.super_rows * a.super_cols * 32 +
                    (int64_t)a.super_rows * 2 * (a.tiles_n - a.super_cols * 16) +
                    rem * ((a.tiles_n + 7) / 8));
    if (a.blocks > 0x7fffffff) return hipErrorInvalidConfiguration;  // past tile_of's 32-bit numbers
    hipLaunchKernelGGL(fused_lse_kernel, grid_of(a.blocks, kThreads), dim3(kThreads), kLdsBytes, stream, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_merge(a, ids, logp_t, flags, stream);
}

}  // namespace stride

extern "C" stride_status stride_debug_fused_band(int32_t band) {
#ifdef STRIDE_FUSED_BAND_HOOK
    if (band < 0) return STRIDE_ERR_INVALID_ARG;
    stride::g_band_override.store(band);
    return STRIDE_OK;
#else
    (void)band;
    return STRIDE_ERR_UNSUPPORTED;
#endif
}
