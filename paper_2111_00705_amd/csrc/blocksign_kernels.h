// Scaled-sign compression per contiguous block (Appendix A, "Scaled sign"), with error feedback
// (Section 4), the server average and the AMSGrad update (Section 3).
//
// The error memory is kept in deferred form.  After a step the library stores x_i = g_i + e_i (the
// vector that was compressed) together with that step's block scales s_i; the error itself,
//     e_i[j] = fl32( x_i[j] - copysign(s_i[block(j)], x_i[j]) ),
// is formed on the fly when the next step (or a getter) reads x_i.  The arithmetic is exactly the
// one of the definition, but one step needs a single pass over g and the stored vector:
//
//   bs_pass     per (tile of 4096 coordinates, worker): e = stored x minus its sign compression
//               (previous scales), x = g + e, store x, write the sign bits of x (1 bit per
//               coordinate), fp64 partial sums of |x| per piece (tile x block); a block that lies
//               inside one tile of several pieces gets its scale here
//   bs_scale    per (other block, worker): fixed-order fp64 sum of the pieces, s = fl32(S / block
//               length) (skipped when every tile lies in one block of at most 8 pieces: bs_update
//               then adds the pieces itself)
//   bs_update   per tile: gbar[j] = (sum_i +-s_i[block(j)]) / n, signs from the stored bits, workers
//               in ascending order; then the AMSGrad update of theta, m, v, vhat
//
// Traffic per (worker, coordinate): 4 B g + 4 B stored x read + 4 B x written + 2 x 1/8 B of sign
// bits, for any block size; plus 32 B per coordinate of optimiser state.
//
// CD-Adam (Section 5, Algorithm 1) runs on the same kernels.  The worker's Markov sequence ghat_i
// takes the place of the error memory, again in deferred form: the library stores ghat_i of the step
// before, and c_i = copysign(s_i[block], sign bit) is added when the next step (or a getter) reads
// it.  The sign bits of c_i cannot be read off the stored vector here, so the step reads the old
// sign word before it writes the new one.
//
//   bs_pass<.., kBsCd>   ghat_i += pending c_i, u = g - ghat_i, store ghat_i, sign bits and piece sums of u
//   bs_scale             as above
//   bs_server            mean of the c_i as above, ghat += mean, w = ghat - gtilde, sign bits and piece
//                        sums of w (the server's compression, lines 8-9 of Algorithm 1)
//   bs_scale             once more, for the single vector w
//   bs_apply             gtilde += copysign(s, w), then the AMSGrad update with gtilde
//
// Traffic: 12 B per (worker, coordinate) as above, plus 12 B + 40 B per coordinate.
#pragma once
#include "device_utils.h"

namespace cams {

// Block table on the device.  A "piece" is the intersection of one block with one 4096-aligned
// tile; pieces are numbered in coordinate order, so the pieces of a tile and the pieces of a
// block are both contiguous ranges.
struct BsTable {
    const int32_t *offsets;      // [n_blocks+1] block boundaries
    const int32_t *piece_hi;     // [n_pieces]   one past the last coordinate of a piece
    const int32_t *piece_blk;    // [n_pieces]   block of a piece
    const int32_t *tile_piece0;  // [n_tiles+1]  first piece of a tile
    const int32_t *block_piece0; // [n_blocks+1] first piece of a block
    int32_t n_blocks;
    int32_t n_pieces;
    int32_t uniform_tiles;       // >0: every block spans this many whole tiles (the last block may be shorter),
                                 // so tile t is piece t of block t / uniform_tiles: no table look-ups needed
    int32_t stream_rows;         // the stored rows are too large to stay cached between steps: bs_pass loads them as a stream
    const int32_t *scale_list;   // [n_scale_list] the blocks whose scale bs_scale forms from the piece sums: all but
    int32_t n_scale_list;        // those that lie inside one tile next to other pieces (bs_pass writes their scale)
    int32_t xcd_chunk;           // bs_pass: tile_of_block's chunk
    int32_t small_log2;          // > 0: uniform blocks of 2^small_log2 coordinates, 4 <= 2^small_log2 < kTile (short blocks)
};

// Short blocks.  With uniform blocks of a power of two below a tile a float4 lies inside one block, whose number is a shift
// of the coordinate, and a block's float4 sit in consecutive lanes of one row r of the tile (or in consecutive rows):
// the sum of |x| is a butterfly in registers, up to 256 coordinates inside one wavefront, and the block's scale is
// complete in the workgroup of its tile.  No table, no staging in LDS, no bs_scale; on small vectors the whole step is one launch
// with blocks of up to 256 (bs_step_short).  Step plus get_theta, n = 16,
// d = 11.2 M, general way / this one, us: error feedback B = 16 660 / 507, B = 256 483 / 476, B = 2048 540 / 476; CD-Adam
// B = 16 810 / 510, B = 1024 606 / 540; n = 20, d = 300, B = 16 under CD-Adam 43 / 24.
constexpr int kSmallMinLog2 = 2, kSmallMaxLog2 = 11;      // 4 .. 2048 coordinates

// Sums of |x| over the block of each row's float4 of this thread, fp64 in a fixed order: S[r] for the block that holds the
// coordinates 4 (tid + 256 r) .. + 3 of the tile (padding holds 0).  part: 16 doubles of LDS.  All threads of the
// workgroup call this; contains a barrier for blocks of more than 256 coordinates.
__device__ __forceinline__ void small_block_sums(const float (&x)[4][4], int log2_len, double (&S)[4], double *part)
{
#pragma unroll
    for (int r = 0; r < 4; ++r)
        S[r] = ((double)fabsf(x[r][0]) + (double)fabsf(x[r][1])) + ((double)fabsf(x[r][2]) + (double)fabsf(x[r][3]));
    const int lanes = 1 << min(log2_len - 2, 6);
    for (int off = 1; off < lanes; off <<= 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) S[r] += __shfl_xor(S[r], off, kWave);
    }
    if (log2_len <= 8) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) part[r * 4 + wave] = S[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (log2_len == 9) {
            S[r] = part[r * 4 + (wave & 2)] + part[r * 4 + (wave & 2) + 1];
        } else {
            const double row = ((part[r * 4] + part[r * 4 + 1]) + part[r * 4 + 2]) + part[r * 4 + 3];
            S[r] = row;
        }
    }
    if (log2_len == 11) {
        S[0] = S[1] = S[0] + S[1];
        S[2] = S[3] = S[2] + S[3];
    }
}

// 2^-k, k below 1023: the product with it is the quotient by 2^k (sums of magnitudes of fp32 are far from fp64's subnormals).
__device__ __forceinline__ double inverse_power(int k) { return __longlong_as_double((long long)(1023 - k) << 52); }

// The scale of the short block (at most 256 coordinates: inside a wavefront's row) that holds the float4 x at coordinate j, in
// every lane of the block; the sums in small_block_sums' order.
__device__ __forceinline__ float short_block_scale(const float (&x)[4], const BsTable &tb, int64_t d, int64_t j)
{
    double S = ((double)fabsf(x[0]) + (double)fabsf(x[1])) + ((double)fabsf(x[2]) + (double)fabsf(x[3]));
    const int lanes = 1 << (tb.small_log2 - 2);
    for (int off = 1; off < lanes; off <<= 1) S += __shfl_xor(S, off, kWave);
    const int64_t len = (int64_t)1 << tb.small_log2;
    const int64_t first = j & ~(len - 1);
    if (__all(first + len <= d)) return (float)(S * inverse_power(tb.small_log2));
    return (float)(S / (double)max((int64_t)1, min(len, d - first)));
}

// Sign bits: per worker, per tile, one 16-bit word per thread of the workgroup.  Bit r*4 + c of
// word `tid` is the sign of the coordinate  tile*4096 + 4*(tid + 256*r) + c,  i.e. of the c-th
// component of the r-th float4 that thread tid handles in the tile (same mapping in bs_pass and
// bs_update).
constexpr int kMaxFusedPieces = 8;   // bs_update adds up to this many pieces of a block itself
constexpr unsigned kPassTileLds = kTile * (sizeof(float) + sizeof(uint16_t));   // dynamic LDS bs_pass needs for a
                                                                                // tile of several pieces

__device__ __forceinline__ float deferred_sign_error(float xs, float s_prev)
{
    return fsub(xs, copysignf(s_prev, xs));
}

// copysign(s, x) for the coordinate whose sign is bit `k` of `bits`; s >= 0.
__device__ __forceinline__ float signed_scale(float s, uint32_t bits, int k)
{
    return __uint_as_float(__float_as_uint(s) | ((bits << (31 - k)) & 0x80000000u));
}

// The pieces of a tile of several pieces, in LDS: bound[q] = end of piece p0 + q relative to the tile
// (1 .. 4096), q < p1 - p0.  Inside a tile consecutive pieces belong to consecutive blocks (a new piece starts
// where a block ends), so the block of piece p0 + q is piece_blk[p0] + q and no table is read per coordinate.
// Ends with a barrier.
__device__ __forceinline__ void stage_piece_bounds(uint16_t *bound, int p0, int p1, const BsTable &tb, int64_t base)
{
    for (int q = threadIdx.x; q < p1 - p0; q += kThreads) bound[q] = (uint16_t)(tb.piece_hi[p0 + q] - (int)base);
    __syncthreads();
}
// Index of the piece that holds coordinate l of the tile: the first q with l < bound[q], the last piece for the
// padding past d.  P >= 1 pieces.
__device__ __forceinline__ int piece_index(const uint16_t *bound, int P, int l)
{
    int lo = 0, hi = P - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (l < (int)bound[mid]) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Fixed-order fp64 sums of |x| over the pieces p0 .. p1-1 of the tile at `base`, one result per piece written
// to out[p].  x: the 16 values of this thread (padding holds 0).
// A tile that is one piece is summed by the whole workgroup.  A tile of several pieces stages |x| in LDS in
// coordinate order (absx, kTile floats) and sums 16 pieces at a time, each by a team of 16 lanes (strided
// partial sums, then a fixed butterfly) - one workgroup reduction per piece made tiles of many short blocks
// tens of times slower.  scales_row (may be null): a block that is a single piece of such a tile lies inside
// the tile, so its scale is complete here and is written at once (bs_scale does not visit it).
// bound: the tile's piece ends as stage_piece_bounds leaves them (only read for a tile of several pieces).
__device__ __forceinline__ void piece_sums(const float (&x)[4][4], int64_t base, int p0, int p1, const BsTable &tb,
                                           double *scratch, float *absx, const uint16_t *bound,
                                           double *__restrict__ out, float *scales_row)
{
    const int tid = threadIdx.x;
    if (p1 - p0 == 1) {
        double acc = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc += (double)fabsf(x[r][c]);
        const double S = block_sum(acc, scratch);
        if (tid == 0) out[p0] = S;
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
        st4(absx + 4 * (tid + kThreads * r), make_float4(fabsf(x[r][0]), fabsf(x[r][1]), fabsf(x[r][2]), fabsf(x[r][3])));
    __syncthreads();
    constexpr int kTeam = 16;
    const int team = tid / kTeam, tl = tid % kTeam;
    const int b0 = tb.piece_blk[p0];
    for (int pb = p0; pb < p1; pb += kThreads / kTeam) {          // uniform over the workgroup
        const int p = pb + team;
        double acc = 0.0;
        int lo = 0, hi = 0;
        if (p < p1) {
            lo = (p == p0) ? 0 : (int)bound[p - p0 - 1];
            hi = (int)bound[p - p0];
            for (int j = lo + tl; j < hi; j += kTeam) acc += (double)absx[j];
        }
#pragma unroll
        for (int off = kTeam / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWave);   // stays inside the team
        if (p < p1 && tl == 0) {
            out[p] = acc;
            if (scales_row) {
                // a piece between two others is a whole block; the first and the last may be parts of longer ones
                const int b = b0 + (p - p0);
                const bool inner = p > p0 && p + 1 < p1;
                if (inner || tb.block_piece0[b + 1] - tb.block_piece0[b] == 1) scales_row[b] = (float)(acc / (double)(hi - lo));
            }
        }
    }
}

// kMode: kBsEf error feedback; kBsCd CD-Adam's worker stage (see the head of this file); kBsNaive naive
// compression (Section 4): x = g, nothing is read from or written to the stored rows.
enum { kBsEf = 0, kBsCd = 1, kBsNaive = 2 };

// G: element type of the gradients, float or uint16_t (bfloat16 bits).
// kSmall: short blocks (BsTable::small_log2); partial is not used then.
template <bool kPending, int kMode, bool kSmall, typename G>
__global__ __launch_bounds__(kThreads) void bs_pass(const G *__restrict__ g, float *__restrict__ xs,
                                                    int64_t d, int64_t ld, BsTable tb,
                                                    float *scales,          // [n][n_blocks]: the previous step's are
                                                                            // read; blocks inside a tile get their new one
                                                    uint16_t *__restrict__ signs,
                                                    double *__restrict__ partial)
{
    __shared__ double scratch[kSmall ? 16 : 4];
    // dynamic LDS, kPassTileLds bytes when the table has tiles of several pieces (only those use it): the staged
    // |x| and the piece ends.  The host may ask for more: the amount also sets how many workgroups share a
    // compute unit, which this kernel is sensitive to (see pass_lds_bytes in the host code).
    extern __shared__ __align__(16) unsigned char pass_lds[];
    float *absx = reinterpret_cast<float *>(pass_lds);
    uint16_t *bound = reinterpret_cast<uint16_t *>(pass_lds + kTile * sizeof(float));
    const float *s_prev = scales;
    const int t = tile_of_block(blockIdx.x, tb.xcd_chunk);
    if (t >= (int)(ld / kTile)) return;
    const int i = blockIdx.y;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)t * kTile;
    const G *grow = g + (int64_t)i * d;
    float *xrow = xs + (int64_t)i * ld;
    const bool uni = kSmall || tb.uniform_tiles > 0;
    const int p0 = uni ? t : tb.tile_piece0[t], p1 = uni ? t + 1 : tb.tile_piece0[t + 1];
    const float *sp = s_prev + (int64_t)i * tb.n_blocks;

    GradRaw<G> gv[4];
    float4 xv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        // The stored row goes first, except with short blocks.  The pass alone, n = 16, d = 11.2 M, gradients first / row first,
        // us: blocks of 100 400 / 396, 200 385 / 380, 1000 374 / 367, bf16 blocks of 100 415 / 408; 62 layers, n = 8 188.5 / 186.7;
        // short blocks of 16 371 / 380, of 256 353 / 360
        // (ld4_row<kSmall>: with short blocks the compiler had merged the two kinds of row load, and rows that should stream were
        // read through the caches; n = 16, d = 11.2 M, step plus get_theta, us, merged / apart: blocks of 256 462 / 429, bf16
        // 412 / 377, of 16 488 / 454, bf16 436 / 400.  Rows that stay cached do not notice the branch: n = 16, d = 1.2 M 64.9 / 64.5 and
        // 66.7 / 66.7, n = 8, d = 1 M 42.1 / 41.9 and 42.2 / 42.0, n = 4, d = 100 000 23.3 / 23.4 and 23.1 / 23.1)
        if (kSmall) gv[r] = load_raw4<false>(grow, j, d);
        xv[r] = kMode == kBsNaive ? make_float4(0.f, 0.f, 0.f, 0.f) : ld4_row<kSmall>(xrow + j, tb.stream_rows);
        if (!kSmall) gv[r] = load_raw4<false>(grow, j, d);
    }
    uint16_t *word = signs + ((int64_t)i * (ld / kTile) + t) * kThreads + tid;
    const uint32_t old_bits = (kMode == kBsCd && kPending) ? (uint32_t)*word : 0u;   // sign bits of the pending c_i
    float x[4][4];
    uint32_t sign_bits = 0;
    const bool single = (p1 - p0 == 1);
    const int P = p1 - p0;
    const int b0 = (uni || (single && !kPending)) ? 0 : tb.piece_blk[p0];     // block of the tile's first piece
    float s_single = (!kSmall && kPending && single) ? sp[uni ? t / tb.uniform_tiles : b0] : 0.f;
    float s_row[4] = {0.f, 0.f, 0.f, 0.f};          // kSmall: the pending scale of each row's float4
    if (kSmall && kPending) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            s_row[r] = sp[min((int)((base + 4 * (tid + kThreads * r)) >> tb.small_log2), tb.n_blocks - 1)];
    }
    if (!single) stage_piece_bounds(bound, p0, p1, tb, base);               // uniform over the workgroup
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        const int l0 = 4 * (tid + kThreads * r);
        const float4 g4 = widen4(gv[r]);
        const float gg[4] = {g4.x, g4.y, g4.z, g4.w};
        const float xx[4] = {xv[r].x, xv[r].y, xv[r].z, xv[r].w};
        float keep[4];     // what goes back to the stored vector
        if (kSmall) s_single = s_row[r];
        int q = (kPending && !single) ? piece_index(bound, P, l0) : 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float s = s_single;
            if (kPending && !single) {
                while (q + 1 < P && l0 + c >= (int)bound[q]) ++q;
                s = sp[b0 + q];
            }
            if (kMode == kBsCd) {
                // ghat_i = ghat_i + c_i (Algorithm 1, line 6, of the step before); u = g - ghat_i (line 5)
                float gh = xx[c];
                if (kPending && j + c < d) gh = fadd(gh, signed_scale(s, old_bits, r * 4 + c));
                keep[c] = gh;
                x[r][c] = (j + c < d) ? fsub(gg[c], gh) : 0.f;
            } else if (kMode == kBsNaive) {
                x[r][c] = (j + c < d) ? gg[c] : 0.f;
                keep[c] = 0.f;
            } else {
                const float e = kPending ? deferred_sign_error(xx[c], s) : xx[c];
                x[r][c] = (j + c < d) ? fadd(gg[c], e) : 0.f;
                keep[c] = x[r][c];
            }
        }
        if (kMode != kBsNaive) st4_stream(xrow + j, make_float4(keep[0], keep[1], keep[2], keep[3]));
#pragma unroll
        for (int c = 0; c < 4; ++c) sign_bits |= (__float_as_uint(x[r][c]) >> 31) << (r * 4 + c);
    }
    *word = (uint16_t)sign_bits;
    if constexpr (kSmall) {
        // a block's scale is rewritten by its first lane, after the block's own lanes have used the old one: they are in
        // the same wavefront, or the barrier inside lies between
        double S[4];
        small_block_sums(x, tb.small_log2, S, scratch);
        const int64_t len = (int64_t)1 << tb.small_log2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t j = base + 4 * (tid + kThreads * r);
            if ((j & (len - 1)) == 0 && j < d)
                scales[(int64_t)i * tb.n_blocks + (j >> tb.small_log2)] = (float)(S[r] / (double)min(len, d - j));
        }
        return;
    }
    // every thread has read the scales it needs (the loop above) before any is rewritten (after the barrier inside)
    piece_sums(x, base, p0, p1, tb, scratch, absx, bound, partial + (int64_t)i * tb.n_pieces,
               scales + (int64_t)i * tb.n_blocks);
}

// One workgroup per (listed block, worker): see BsTable::scale_list.  One wavefront adds the block's pieces, lane l
// those at l, l + 64, ..., and a fixed butterfly follows: the order does not depend on the launch shape.
// Bound by latency.  A block of at most kDirectPieces pieces is added straight from memory.  A longer one (the
// whole-vector sign of 11.2 M coordinates has 2728 pieces, of 110 M 26 856) is staged in LDS by a workgroup of
// kThreads, kScaleStage pieces at a time with the next ones in flight: one wavefront alone waits for memory once in
// 64 pieces.
constexpr int kDirectPieces = 256;
constexpr int kScaleStage = 2048;
constexpr int kStagePer = kScaleStage / kThreads;
__global__ __launch_bounds__(kThreads) void bs_scale(const double *__restrict__ partial, BsTable tb,
                                                     float *__restrict__ scales)
{
    // dynamic LDS: kScaleStage doubles when some block is long (launched with kThreads), else none
    extern __shared__ __align__(16) unsigned char scale_lds[];
    double *stage = reinterpret_cast<double *>(scale_lds);
    const int b = tb.scale_list[blockIdx.x];
    const int i = blockIdx.y;
    const int tid = threadIdx.x;
    const int q0 = tb.block_piece0[b], q1 = tb.block_piece0[b + 1];
    const double *row = partial + (int64_t)i * tb.n_pieces;
    double acc = 0.0;
    if (q1 - q0 <= kDirectPieces || blockDim.x < kThreads) {
        if (tid >= kWave) return;
        for (int q = q0 + tid; q < q1; q += kWave) acc += row[q];
    } else {
        double next[kStagePer];
#pragma unroll
        for (int u = 0; u < kStagePer; ++u) {
            const int q = q0 + u * kThreads + tid;
            next[u] = q < q1 ? row[q] : 0.0;
        }
        for (int base = q0; base < q1; base += kScaleStage) {
            __syncthreads();                                   // the stage has been added up
#pragma unroll
            for (int u = 0; u < kStagePer; ++u) stage[u * kThreads + tid] = next[u];
#pragma unroll
            for (int u = 0; u < kStagePer; ++u) {
                const int q = base + kScaleStage + u * kThreads + tid;
                next[u] = q < q1 ? row[q] : 0.0;
            }
            __syncthreads();
            if (tid < kWave) {
                const int cnt = min(kScaleStage, q1 - base);
#pragma unroll 8
                for (int q = tid; q < cnt; q += kWave) acc += stage[q];
            }
        }
        if (tid >= kWave) return;
    }
    const double S = wave_sum(acc);
    if (tid == 0) {
        const double len = (double)(tb.offsets[b + 1] - tb.offsets[b]);
        scales[(int64_t)i * tb.n_blocks + b] = (float)(S / len);
    }
}

constexpr int kScaleChunk = 1024;   // workers whose scales are staged in LDS at a time
constexpr int kSignBatch = 8;       // workers whose sign words are loaded together

// CD-Adam's server stage (Algorithm 1, lines 8-9): the mean of the c_i goes into ghat, w = ghat - gtilde is formed, and
// its sign bits and piece sums are written for the second compression.  One workgroup per tile: a piece of w is summed
// by the workgroup that holds all of it.  kFusedScale: every tile lies inside one block of at most kMaxFusedPieces
// pieces; the workers' scales are then formed here from the partial sums (and stored by the tile at the block's
// start).  kStreamState: theta, m, v, vhat (touched only with whole_blocks) and ghat, which nothing else in a step reads, are
// loaded and stored as streams; gtilde, which bs_apply reads again, is left cached until its own last store.  (Whole-vector
// sign, step plus get_theta: n = 8, d = 11.2 M 336.5 -> 331.8 us, n = 2, d = 60 M bf16 877 -> 831; blocks of 4096, n = 8,
// d = 8 M 236 -> 226.)
struct BsMarkov {
    float *ghat;            // [ld] the server's aggregate
    float *gtil;            // [ld] gtilde of the step before (rewritten here only when whole_blocks is set)
    uint16_t *signs;        // [n_tiles][256] sign bits of w
    double *partial;        // [n_pieces] piece sums of |w|
    float *scales;          // [n_blocks] scales of the server's message
    int32_t whole_blocks;   // every tile is exactly one block: the block's scale of w is known inside the
                            // workgroup, so lines 9-16 of Algorithm 1 follow at once (no bs_scale, no bs_apply).  Set
                            // where kFusedScale is; known at compile time, with the LDS that such tiles do not need left
                            // out, bs_server took longer (blocks of 4096, n = 8, d = 8 M 68.4 -> 72.1 us)
};

template <bool kFusedScale, bool kStreamState>
__global__ __launch_bounds__(kThreads) void bs_server(int64_t d, int64_t ld, int n, BsTable tb,
                                                      const double *__restrict__ partial,
                                                      float *__restrict__ scales,
                                                      const uint16_t *__restrict__ signs,
                                                      float *__restrict__ theta, float *__restrict__ m,
                                                      float *__restrict__ v, float *__restrict__ vhat, AmsParams p,
                                                      BsMarkov mk)
{
    __shared__ float s_lds[kScaleChunk];
    __shared__ double scratch[4];
    __shared__ float absx[kTile];                    // piece_sums of the server's vector
    __shared__ uint16_t bound[kTile];                // piece ends of a tile where several blocks meet
    const int t = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)t * kTile;
    const int n_tiles = (int)(ld / kTile);

    float acc[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.f;
    const uint16_t *srow = signs + (int64_t)t * kThreads + tid;
    const int64_t sstride = (int64_t)n_tiles * kThreads;

    // sign words of the first workers go out before anything waits
    uint32_t bits[kSignBatch];
#pragma unroll
    for (int u = 0; u < kSignBatch; ++u) bits[u] = (u < n) ? srow[u * sstride] : 0u;

    int p0, p1, b_single;
    if (tb.uniform_tiles > 0) {
        p0 = t;
        p1 = t + 1;
        b_single = t / tb.uniform_tiles;
    } else {
        p0 = tb.tile_piece0[t];
        p1 = tb.tile_piece0[t + 1];
        b_single = tb.piece_blk[p0];
    }
    const bool single = kFusedScale || (p1 - p0 == 1);

    if (single) {
        int q0 = 0, q1 = 0;
        double len = 1.0;
        if (kFusedScale) {
            if (tb.uniform_tiles > 0) {
                q0 = b_single * tb.uniform_tiles;
                q1 = min(q0 + tb.uniform_tiles, n_tiles);
                len = (double)min((int64_t)tb.uniform_tiles * kTile, d - (int64_t)q0 * kTile);
            } else {
                q0 = tb.block_piece0[b_single];
                q1 = tb.block_piece0[b_single + 1];
                len = (double)(tb.offsets[b_single + 1] - tb.offsets[b_single]);
            }
        }
        for (int c0 = 0; c0 < n; c0 += kScaleChunk) {
            const int cn = min(kScaleChunk, n - c0);
            __syncthreads();
            // one thread per worker: the scale of this tile's block
            for (int u = tid; u < cn; u += kThreads) {
                const int i = c0 + u;
                float s;
                if (kFusedScale) {
                    const double *prow = partial + (int64_t)i * tb.n_pieces;
                    double S = 0.0;
                    for (int q = q0; q < q1; ++q) S += prow[q];
                    s = (float)(S / len);
                    if (q0 == p0) scales[(int64_t)i * tb.n_blocks + b_single] = s;   // this tile starts the block
                } else {
                    s = scales[(int64_t)i * tb.n_blocks + b_single];
                }
                s_lds[u] = s;
            }
            __syncthreads();
            for (int u0 = 0; u0 < cn; u0 += kSignBatch) {
                // the sign words of the batch after this one go out before this one is used
                uint32_t next[kSignBatch];
                const int w1 = c0 + u0 + kSignBatch;       // first worker of the next batch (may be in the next chunk)
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) next[u] = (w1 + u < n) ? srow[(w1 + u) * sstride] : 0u;
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) {
                    if (u0 + u < cn) {
                        const float s = s_lds[u0 + u];
#pragma unroll
                        for (int q = 0; q < 16; ++q) acc[q] = fadd(acc[q], signed_scale(s, bits[u], q));
                    }
                }
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) bits[u] = next[u];
            }
        }
    } else {
        // several blocks meet in this tile: find the block of every coordinate
        stage_piece_bounds(bound, p0, p1, tb, base);
        const int P = p1 - p0;
        int blk[16];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int l0 = 4 * (tid + kThreads * r);
            int q = piece_index(bound, P, l0);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                while (q + 1 < P && l0 + c >= (int)bound[q]) ++q;
                blk[r * 4 + c] = b_single + q;            // b_single: the block of the tile's first piece
            }
        }
        for (int i = 0; i < n; ++i) {
            const uint32_t w = srow[i * sstride];
            const float *sc = scales + (int64_t)i * tb.n_blocks;
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[q] = fadd(acc[q], signed_scale(sc[blk[q]], w, q));
        }
    }
    float w[4][4];
    uint32_t sign_bits = 0;
    // All four rows' loads go out before the first row is stored, and below the next row's state before a row is stored: the
    // compiler does not take a load past a store that might write what it reads, and a workgroup waited for memory row by
    // row.  Step plus get_theta, us, before / after: whole-vector sign n = 8, d = 11.2 M 319.6 / 317.6, n = 4, d = 30 M bf16 539 /
    // 532, 62 layers n = 8 bf16 310.6 / 306.6, blocks of 4096 n = 8, d = 8 M 219.5 / 216.2, n = 4, d = 60 000 28.4 / 27.8.  The
    // one-launch form pays for it with 104 registers instead of 77, four wavefronts per SIMD instead of five.
    float4 gh_row[4], gt_row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        gh_row[r] = ld4_state<kStreamState>(mk.ghat + j);
        gt_row[r] = ld4(mk.gtil + j);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        const float4 gh4 = gh_row[r], gt4 = gt_row[r];
        const float gh[4] = {gh4.x, gh4.y, gh4.z, gh4.w}, gt[4] = {gt4.x, gt4.y, gt4.z, gt4.w};
        float nh[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            // padding coordinates stay 0
            nh[c] = (j + c < d) ? fadd(gh[c], fdiv(acc[r * 4 + c], p.n_workers)) : gh[c];
            w[r][c] = (j + c < d) ? fsub(nh[c], gt[c]) : 0.f;
            sign_bits |= (__float_as_uint(w[r][c]) >> 31) << (r * 4 + c);
        }
        st4_state<kStreamState>(mk.ghat + j, make_float4(nh[0], nh[1], nh[2], nh[3]));
    }
    mk.signs[(int64_t)t * kThreads + tid] = (uint16_t)sign_bits;
    __syncthreads();   // s_lds readers are done before scratch is used (separate arrays; keeps phases apart)
    if (!mk.whole_blocks) {
        piece_sums(w, base, p0, p1, tb, scratch, absx, bound, mk.partial, mk.scales);
        return;
    }
    // c = C(w) with the scale of this tile's block, gtilde += c, AMSGrad with gtilde
    double a64 = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) a64 += (double)fabsf(w[r][c]);
    const double S = block_sum(a64, scratch);
    const double blen = (double)min((int64_t)kTile, d - base);
    const float s = (float)(S / blen);
    if (tid == 0) mk.scales[b_single] = s;
    const int64_t j0 = base + 4 * tid;
    float4 th = ld4_state<kStreamState>(theta + j0), mm = ld4_state<kStreamState>(m + j0), vv = ld4_state<kStreamState>(v + j0),
           vh = ld4_state<kStreamState>(vhat + j0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        const float4 gt4 = gt_row[r];
        const float gt[4] = {gt4.x, gt4.y, gt4.z, gt4.w};
        float nt[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            nt[c] = (j + c < d) ? fadd(gt[c], signed_scale(s, sign_bits, r * 4 + c)) : gt[c];   // padding stays 0
        const float4 g4 = make_float4(nt[0], nt[1], nt[2], nt[3]);
        float4 th4 = th, m4 = mm, v4 = vv, vh4 = vh;
        if (r < 3) {                                  // the next row's, before this one is stored
            th = ld4_state<kStreamState>(theta + j + 4 * kThreads);
            mm = ld4_state<kStreamState>(m + j + 4 * kThreads);
            vv = ld4_state<kStreamState>(v + j + 4 * kThreads);
            vh = ld4_state<kStreamState>(vhat + j + 4 * kThreads);
        }
        amsgrad_update4(th4, m4, v4, vh4, g4, p);
        st4_state<kStreamState>(mk.gtil + j, g4);
        st4_state<kStreamState>(theta + j, th4);
        st4_state<kStreamState>(m + j, m4);
        st4_state<kStreamState>(v + j, v4);
        st4_state<kStreamState>(vhat + j, vh4);
    }
}

// Lines 8-12 of Algorithm 1 for short blocks inside a wavefront: gb, the mean of the c_i on the float4 at coordinate j, becomes
// gtilde; ghat, gtilde and the server's scales are written.  gh4, gt4: ghat and gtilde there; blk: the float4's block.  Returns
// the sign bits of the server's vector.
template <bool kStreamState>
__device__ __forceinline__ uint32_t short_server(float (&gb)[4], const float4 &gh4, const float4 &gt4, const BsMarkov &mk,
                                                 const BsTable &tb, int64_t d, int64_t j, int blk)
{
    const float gh[4] = {gh4.x, gh4.y, gh4.z, gh4.w}, gt[4] = {gt4.x, gt4.y, gt4.z, gt4.w};
    float nh[4], w[4];
    uint32_t neg = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        nh[c] = (j + c < d) ? fadd(gh[c], gb[c]) : gh[c];          // padding coordinates stay 0
        w[c] = (j + c < d) ? fsub(nh[c], gt[c]) : 0.f;
        neg |= (__float_as_uint(w[c]) >> 31) << c;
    }
    st4_state<kStreamState>(mk.ghat + j, make_float4(nh[0], nh[1], nh[2], nh[3]));
    const float s = short_block_scale(w, tb, d, j);
    if ((j & (((int64_t)1 << tb.small_log2) - 1)) == 0 && j < d) mk.scales[blk] = s;
#pragma unroll
    for (int c = 0; c < 4; ++c) gb[c] = (j + c < d) ? fadd(gt[c], signed_scale(s, neg, c)) : gt[c];   // gtilde
    st4_state<kStreamState>(mk.gtil + j, make_float4(gb[0], gb[1], gb[2], gb[3]));
    return neg;
}

// Server average and AMSGrad update, a quarter of a tile per workgroup, one float4 per thread.  Workgroup 4 t + w takes the
// words of the threads 64 w .. 64 w + 63 of tile t, wavefront r of it their nibble r, so the four wavefronts share the
// sign words they read.  With one float4 the registers leave room for many wavefronts, and the sign words (and scales)
// of eight workers are in flight together.  HBM-bound where the vector is long (32 B per coordinate, n/8 B of signs),
// latency-bound below a million coordinates.
// kBlocks: where a float4's scales come from -
//   kBlocksShort  short blocks (BsTable::small_log2): one scale per float4
//   kBlocksFused  every tile lies inside one block of at most kMaxFusedPieces pieces: the scale is formed here from the
//                 piece sums (and stored by the tile at the block's start)
//   kBlocksTable  any table: one scale where the tile lies inside one block, else one per coordinate
// kEarlyState: theta, m, v, vhat are loaded first (small grids: nothing else would hide that latency).
// theta_out (kBlocksFused; may be null): d floats of the caller's, 4-byte aligned, that receive the new theta as well.
// kMarkov (kBlocksShort with blocks of at most 256 coordinates, which lie inside a wavefront): CD-Adam's server stage,
// lines 8-16 of Algorithm 1 in this one launch (no bs_scale, no bs_apply).
enum { kBlocksShort = 0, kBlocksFused = 1, kBlocksTable = 2 };
template <int kBlocks, bool kEarlyState, bool kMarkov, bool kStreamState>
__global__ __launch_bounds__(kThreads) void bs_update(int64_t d, int64_t ld, int n, BsTable tb,
                                                      const double *__restrict__ partial, float *__restrict__ scales,
                                                      const uint16_t *__restrict__ signs,
                                                      float *__restrict__ theta, float *__restrict__ m,
                                                      float *__restrict__ v, float *__restrict__ vhat, AmsParams p,
                                                      BsMarkov mk, float *__restrict__ theta_out)
{
    __shared__ float s_lds[kBlocks == kBlocksFused ? kScaleChunk : 1];
    const int t = blockIdx.x >> 2;
    const int lane = threadIdx.x & 63, r = threadIdx.x >> 6;
    const int slot = (blockIdx.x & 3) * kWave + lane;                       // thread of the tile; r: row
    const int64_t base = (int64_t)t * kTile;
    const int64_t j = base + 4 * (slot + kThreads * r);
    const int n_tiles = (int)(ld / kTile);
    const int64_t sstride = (int64_t)n_tiles * kThreads;
    const uint16_t *srow = signs + (int64_t)t * kThreads + slot;

    float4 th, mm, vv, vh;
    if (kEarlyState) {
        th = ld4_state<kStreamState>(theta + j);
        mm = ld4_state<kStreamState>(m + j);
        vv = ld4_state<kStreamState>(v + j);
        vh = ld4_state<kStreamState>(vhat + j);
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    int blk = 0;                                    // the float4's block (kBlocksShort), the tile's (else)
    if constexpr (kBlocks == kBlocksShort) {
        blk = min((int)(j >> tb.small_log2), tb.n_blocks - 1);
        const float *sc = scales + blk;
        for (int i0 = 0; i0 < n; i0 += kSignBatch) {
            uint32_t bits[kSignBatch];
            float s[kSignBatch];
#pragma unroll
            for (int u = 0; u < kSignBatch; ++u) {
                const int i = min(i0 + u, n - 1);            // clamped: the copies past n are not used
                bits[u] = srow[i * sstride];
                s[u] = sc[(int64_t)i * tb.n_blocks];
            }
#pragma unroll
            for (int u = 0; u < kSignBatch; ++u) {
                if (i0 + u < n) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] = fadd(acc[c], signed_scale(s[u], bits[u] >> (4 * r), c));
                }
            }
        }
    } else if constexpr (kBlocks == kBlocksFused) {
        int q0, q1;
        double len;
        if (tb.uniform_tiles > 0) {
            blk = t / tb.uniform_tiles;
            q0 = blk * tb.uniform_tiles;
            q1 = min(q0 + tb.uniform_tiles, n_tiles);
            len = (double)min((int64_t)tb.uniform_tiles * kTile, d - (int64_t)q0 * kTile);
        } else {
            blk = tb.piece_blk[t];                   // one piece per tile
            q0 = tb.block_piece0[blk];
            q1 = tb.block_piece0[blk + 1];
            len = (double)(tb.offsets[blk + 1] - tb.offsets[blk]);
        }
        for (int c0 = 0; c0 < n; c0 += kScaleChunk) {
            const int cn = min(kScaleChunk, n - c0);
            uint32_t bits[kSignBatch];
#pragma unroll
            for (int u = 0; u < kSignBatch; ++u) bits[u] = srow[min(c0 + u, n - 1) * sstride];   // before the barriers
            if (c0) __syncthreads();
            for (int u = threadIdx.x; u < cn; u += kThreads) {       // one thread per worker: the scale of this tile's block
                const double *prow = partial + (int64_t)(c0 + u) * tb.n_pieces;
                double S = 0.0;
                for (int q = q0; q < q1; ++q) S += prow[q];
                const float s = (float)(S / len);
                if (q0 == t && (blockIdx.x & 3) == 0) scales[(int64_t)(c0 + u) * tb.n_blocks + blk] = s;
                s_lds[u] = s;
            }
            __syncthreads();
            for (int u0 = 0; u0 < cn; u0 += kSignBatch) {
                uint32_t next[kSignBatch];
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) next[u] = srow[min(c0 + u0 + kSignBatch + u, n - 1) * sstride];
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) {
                    if (u0 + u < cn) {
                        const float s = s_lds[u0 + u];
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[c] = fadd(acc[c], signed_scale(s, bits[u] >> (4 * r), c));
                    }
                }
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) bits[u] = next[u];
            }
        }
    } else {
        const int p0 = tb.uniform_tiles > 0 ? t : tb.tile_piece0[t], p1 = tb.uniform_tiles > 0 ? t + 1 : tb.tile_piece0[t + 1];
        blk = tb.uniform_tiles > 0 ? t / tb.uniform_tiles : tb.piece_blk[p0];
        if (p1 - p0 == 1) {
            const float *sc = scales + blk;          // uniform over the workgroup
            for (int i0 = 0; i0 < n; i0 += kSignBatch) {
                uint32_t bits[kSignBatch];
                float s[kSignBatch];
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) {
                    const int i = min(i0 + u, n - 1);
                    bits[u] = srow[i * sstride];
                    s[u] = sc[(int64_t)i * tb.n_blocks];
                }
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) {
                    if (i0 + u < n) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[c] = fadd(acc[c], signed_scale(s[u], bits[u] >> (4 * r), c));
                    }
                }
            }
        } else {
            // several blocks meet in this tile: the piece of each coordinate by binary search over the tile's piece ends
            // (consecutive pieces of a tile belong to consecutive blocks); padding past d takes the last one
            int lo = p0, hi = p1 - 1;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (j < (int64_t)tb.piece_hi[mid]) hi = mid; else lo = mid + 1;
            }
            int at[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                while (lo + 1 < p1 && j + c >= (int64_t)tb.piece_hi[lo]) ++lo;
                at[c] = blk + (lo - p0);
            }
            for (int i0 = 0; i0 < n; i0 += 4) {
                uint32_t bits[4];
                float s[4][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = min(i0 + u, n - 1);
                    bits[u] = srow[i * sstride];
#pragma unroll
                    for (int c = 0; c < 4; ++c) s[u][c] = scales[(int64_t)i * tb.n_blocks + at[c]];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (i0 + u < n) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[c] = fadd(acc[c], signed_scale(s[u][c], bits[u] >> (4 * r), c));
                    }
                }
            }
        }
    }
    // padding coordinates take no gradient
    float gb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) gb[c] = j + c < d ? fdiv(acc[c], p.n_workers) : 0.f;
    if constexpr (kMarkov) {
        const float4 gh4 = ld4_state<kStreamState>(mk.ghat + j), gt4 = ld4_state<kStreamState>(mk.gtil + j);
        // the server's sign words: the four wavefronts hold a nibble each
        __shared__ uint32_t nib[4][kWave];
        nib[r][lane] = short_server<kStreamState>(gb, gh4, gt4, mk, tb, d, j, blk);
        __syncthreads();
        if (r == 0) {
            mk.signs[(int64_t)t * kThreads + slot] =
                (uint16_t)(nib[0][lane] | (nib[1][lane] << 4) | (nib[2][lane] << 8) | (nib[3][lane] << 12));
        }
    }
    if (!kEarlyState) {
        th = ld4_state<kStreamState>(theta + j);
        mm = ld4_state<kStreamState>(m + j);
        vv = ld4_state<kStreamState>(v + j);
        vh = ld4_state<kStreamState>(vhat + j);
    }
    amsgrad_update4(th, mm, vv, vh, make_float4(gb[0], gb[1], gb[2], gb[3]), p);
    st4_state<kStreamState>(theta + j, th);
    if (kBlocks == kBlocksFused && theta_out) {
        // a caller who asked for theta while this update was pending gets it from the registers
        if (j + 4 <= d) {
            const v4f o = {th.x, th.y, th.z, th.w};
            *reinterpret_cast<v4f_any *>(theta_out + j) = o;
        } else {
            if (j < d) theta_out[j] = th.x;
            if (j + 1 < d) theta_out[j + 1] = th.y;
            if (j + 2 < d) theta_out[j + 2] = th.z;
        }
    }
    st4_state<kStreamState>(m + j, mm);
    st4_state<kStreamState>(v + j, vv);
    st4_state<kStreamState>(vhat + j, vh);
}

// A whole step with short blocks of at most 256 coordinates in one launch, for vectors that leave the chip idle (one_launch_sign):
// a quarter of a tile per workgroup, words and coordinates as in bs_update.  Twelve wavefronts share the (row, worker) pairs, each
// with a row of its own; a block lies inside a row, so a worker's scale and sign bits are known where its row was read, and go
// through LDS to four more wavefronts, which add the c_i up in ascending worker order and update the state.
// Bound by latency: the state and kStepBatch pairs of every wavefront are in flight together, one barrier, and nothing waits for a
// store; rows of padding are left out.
// CD-Adam n = 20, d = 300, blocks of 16: bs_pass 4.7 us and bs_update 5.7 with a gap between them, this 6.2; step plus
// get_theta 24.2 -> 20.5.  (Eight workers a wavefront, four rows always and everything unrolled, 9.3 us: its instructions took longer
// to fetch and issue than the loads.)
constexpr int kStepWaves = 12, kStepThreads = (kStepWaves + 4) * kWave;     // 12: a multiple of 1, 2, 3 and 4 rows
constexpr int kStepBatch = 4;
constexpr unsigned kStepLdsPerWorker = kThreads * (sizeof(float) + sizeof(uint8_t));   // dynamic LDS
template <bool kPending, int kMode, typename G, bool kStreamState>
__global__ __launch_bounds__(kStepThreads) void bs_step_short(const G *__restrict__ g, float *__restrict__ xs, int64_t d, int64_t ld,
                                                              int n, BsTable tb, float *__restrict__ scales,
                                                              uint16_t *__restrict__ signs, float *__restrict__ theta,
                                                              float *__restrict__ m, float *__restrict__ v,
                                                              float *__restrict__ vhat, AmsParams p, BsMarkov mk)
{
    constexpr bool kMarkov = kMode == kBsCd;
    extern __shared__ __align__(16) unsigned char step_lds[];
    float (*s_lds)[kThreads] = reinterpret_cast<float (*)[kThreads]>(step_lds);           // [n] a worker's scale for each float4
    uint8_t (*nib)[4][kWave] = reinterpret_cast<uint8_t (*)[4][kWave]>(s_lds + n);        // [n] its sign bits there
    __shared__ uint8_t server_nib[4][kWave];
    const int t = blockIdx.x >> 2;
    const uint32_t lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t quarter = (int64_t)t * kTile + 4 * kWave * (blockIdx.x & 3);
    if (quarter >= d) return;                              // padding: all of it stays 0
    const int rows = (int)min((int64_t)4, (d - quarter + 4 * kThreads - 1) / (4 * kThreads));    // the others are padding
    const bool updates = wave >= kStepWaves;
    // wave / rows and wave % rows without a division; step: wavefronts of a row
    const int of = rows == 1 ? wave : rows == 2 ? wave >> 1 : rows == 3 ? (wave * 11) >> 5 : wave >> 2;
    const int step = rows == 1 ? 12 : rows == 2 ? 6 : rows == 3 ? 4 : 3;
    const int r = updates ? wave - kStepWaves : wave - of * rows;
    const uint32_t at = 4u * (lane + kThreads * r);
    const int64_t j = quarter + at;
    const int64_t sstride = (int64_t)(ld / kTile) * kThreads;
    const int64_t word0 = (int64_t)t * kThreads + (blockIdx.x & 3) * kWave;
    const int blk = min((int)(j >> tb.small_log2), tb.n_blocks - 1);
    auto word = [&](const uint8_t (*q)[kWave]) {
        uint32_t w = q[0][lane];
        if (rows > 1) w |= q[1][lane] << 4;
        if (rows > 2) w |= q[2][lane] << 8;
        if (rows > 3) w |= q[3][lane] << 12;
        return (uint16_t)w;
    };
    if (!updates) {
        const GradPlace place = grad_place(j, d);          // two short blocks at least: d > 4
        const int64_t len64 = (int64_t)1 << tb.small_log2;
        const int64_t first = j & ~(len64 - 1);
        const bool heads = j == first && j < d;            // the block's first float4
        const bool whole = quarter + 4 * kThreads * r + 4 * kWave <= d;       // no block of the row is cut
        const int lanes = 1 << (tb.small_log2 - 2);
        for (int w0 = of; w0 < n; w0 += kStepBatch * step) {
            GradRaw<G> gv[kStepBatch];
            float4 xv[kStepBatch];
            float s_old[kStepBatch];
            uint32_t old_bits[kStepBatch], neg[kStepBatch];
            double S[kStepBatch];
#pragma unroll
            for (int u = 0; u < kStepBatch; ++u) {
                const int i = min(w0 + u * step, n - 1);   // clamped: the copies past n are not used
                gv[u] = load_place4(g + (int64_t)i * d, place);
                xv[u] = kMode == kBsNaive ? make_float4(0.f, 0.f, 0.f, 0.f) : ld4(at_offset(xs + (int64_t)i * ld + quarter, at));
                s_old[u] = kPending ? scales[(int64_t)i * tb.n_blocks + blk] : 0.f;
                old_bits[u] = kMarkov && kPending ? (uint32_t)*at_offset(signs + (int64_t)i * sstride + word0, lane) >> (4 * r) : 0u;
            }
            // stage by stage over the batch: what one worker does is a chain of latencies
#pragma unroll
            for (int u = 0; u < kStepBatch; ++u) {
                const float4 g4 = shift4(widen4(gv[u]), place.shift);
                const float gg[4] = {g4.x, g4.y, g4.z, g4.w};
                const float xx[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
                float x[4], keep[4] = {0.f, 0.f, 0.f, 0.f};
                neg[u] = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool in = j + c < d;
                    if (kMarkov) {
                        const float gh = kPending ? fadd(xx[c], signed_scale(s_old[u], old_bits[u], c)) : xx[c];
                        keep[c] = in ? gh : xx[c];
                        x[c] = in ? fsub(gg[c], gh) : 0.f;
                    } else if (kMode == kBsNaive) {
                        x[c] = in ? gg[c] : 0.f;
                    } else {
                        const float sum = fadd(gg[c], kPending ? deferred_sign_error(xx[c], s_old[u]) : xx[c]);
                        keep[c] = x[c] = in ? sum : 0.f;
                    }
                    neg[u] |= (__float_as_uint(x[c]) >> 31) << c;
                }
                xv[u] = make_float4(keep[0], keep[1], keep[2], keep[3]);
                S[u] = ((double)fabsf(x[0]) + (double)fabsf(x[1])) + ((double)fabsf(x[2]) + (double)fabsf(x[3]));
            }
            for (int off = 1; off < lanes; off <<= 1) {
#pragma unroll
                for (int u = 0; u < kStepBatch; ++u) S[u] += __shfl_xor(S[u], off, kWave);
            }
            if (whole) {
                const double inv = inverse_power(tb.small_log2);
#pragma unroll
                for (int u = 0; u < kStepBatch; ++u) S[u] *= inv;
            } else {
                const double len = (double)max((int64_t)1, min(len64, d - first));
#pragma unroll
                for (int u = 0; u < kStepBatch; ++u) S[u] /= len;
            }
#pragma unroll
            for (int u = 0; u < kStepBatch; ++u) {
                const int i = w0 + u * step;
                if (i < n) {
                    const float s = (float)S[u];
                    s_lds[i][r * kWave + lane] = s;
                    nib[i][r][lane] = (uint8_t)neg[u];
                    if (kMode != kBsNaive) st4_stream(at_offset(xs + (int64_t)i * ld + quarter, at), xv[u]);
                    if (heads) scales[(int64_t)i * tb.n_blocks + blk] = s;
                }
            }
        }
        lds_barrier();
        // the words of the workers in turn; the old ones, which all rows needed, have been read
        for (int i = wave; i < n; i += kStepWaves) *at_offset(signs + (int64_t)i * sstride + word0, lane) = word(nib[i]);
        if (kMarkov) lds_barrier();
        return;
    }
    float4 th, mm, vv, vh, gh4, gt4;
    const bool live = r < rows;
    if (live) {
        th = ld4_state<kStreamState>(theta + j);
        mm = ld4_state<kStreamState>(m + j);
        vv = ld4_state<kStreamState>(v + j);
        vh = ld4_state<kStreamState>(vhat + j);
        if (kMarkov) {
            gh4 = ld4_state<kStreamState>(mk.ghat + j);
            gt4 = ld4_state<kStreamState>(mk.gtil + j);
        }
    }
    lds_barrier();
    float gb[4];
    if (live) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int i = 0; i < n; ++i) {
            const float s = s_lds[i][r * kWave + lane];
            const uint32_t bits = nib[i][r][lane];
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = fadd(acc[c], signed_scale(s, bits, c));
        }
        // padding coordinates take no gradient
#pragma unroll
        for (int c = 0; c < 4; ++c) gb[c] = j + c < d ? fdiv(acc[c], p.n_workers) : 0.f;
        if (kMarkov) server_nib[r][lane] = (uint8_t)short_server<kStreamState>(gb, gh4, gt4, mk, tb, d, j, blk);
    }
    if (kMarkov) {
        lds_barrier();
        if (r == 0) *at_offset(mk.signs + word0, lane) = word(server_nib);
    }
    if (!live) return;
    amsgrad_update4(th, mm, vv, vh, make_float4(gb[0], gb[1], gb[2], gb[3]), p);
    st4_state<kStreamState>(theta + j, th);
    st4_state<kStreamState>(m + j, mm);
    st4_state<kStreamState>(v + j, vv);
    st4_state<kStreamState>(vhat + j, vh);
}

// ---------------------------------------------------------------------------------------------
// Error feedback with uniform blocks of whole tiles (at most kMaxFusedPieces each), one launch per step.
// The AMSGrad update of a step depends on nothing but that step's sign words and piece sums, and the next step's
// pass reads neither theta, m, v nor vhat: so the update of step t is deferred and runs inside the pass kernel of
// step t + 1, as extra workgroups that are dispatched first (blockIdx.y < 4: the four quarters of every tile;
// blockIdx.y >= 4: the pass of worker blockIdx.y - 4).  On small models the update alone is a chain of latencies
// on a mostly idle chip (293 workgroups for 1.2 M coordinates); inside the pass it costs its bytes.  Sign words
// and piece sums exist twice and alternate: the pass of step t + 1 writes one set while the update of step t reads
// the other.  The scales of step t are formed from its piece sums where they are needed - by the pass (the
// deferred error of the stored rows) and by the update - with the same arithmetic: the fp64 sum of the block's
// pieces in coordinate order, one division, one rounding.
struct BsDeferred {
    const uint16_t *signs_prev;     // [n][n_tiles][256] sign words of the step whose update is pending
    const double *partial_prev;     // [n][n_pieces] its piece sums (also what the pass takes the pending scales from)
    float *scales_out;              // [n][n_blocks] the update writes that step's scales here (for the getters)
    float *theta, *m, *v, *vhat;
    AmsParams p;                    // hyper-parameters of the step whose update is pending
    int32_t do_update;              // 0: nothing is pending (first step, or the update has been run on its own)
};

// The scale of block b = the tile's block for worker i from that worker's piece sums (uniform tiles).
__device__ __forceinline__ float fused_block_scale(const double *__restrict__ prow, int b, const BsTable &tb, int n_tiles,
                                                   int64_t d)
{
    const int q0 = b * tb.uniform_tiles, q1 = min(q0 + tb.uniform_tiles, n_tiles);
    const double len = (double)min((int64_t)tb.uniform_tiles * kTile, d - (int64_t)q0 * kTile);
    double S = 0.0;
    for (int q = q0; q < q1; ++q) S += prow[q];
    return (float)(S / len);
}

template <bool kPending, typename G, bool kStreamState>
__global__ __launch_bounds__(kThreads) void bs_pass_update(const G *__restrict__ g, float *__restrict__ xs, int64_t d,
                                                           int64_t ld, int n, BsTable tb,
                                                           uint16_t *__restrict__ signs, double *__restrict__ partial,
                                                           BsDeferred df)
{
    __shared__ double scratch[4];
    __shared__ float s_lds[kScaleChunk];
    // dynamic LDS: none is used; the amount only sets how many workgroups share a compute unit (see bs_pass)
    const int n_tiles = (int)(ld / kTile);
    const int t = tile_of_block(blockIdx.x, tb.xcd_chunk);
    if (t >= n_tiles) return;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)t * kTile;
    const int b = t / tb.uniform_tiles;

    if (blockIdx.y < 4) {
        // ---- the pending update of quarter r of tile t: coordinates base + 4 (tid + 256 r) + c
        if (!df.do_update) return;
        const int r = blockIdx.y;
        const int64_t j = base + 4 * (tid + kThreads * r);
        const float4 th0 = ld4_state<kStreamState>(df.theta + j), m0 = ld4_state<kStreamState>(df.m + j),
                     v0 = ld4_state<kStreamState>(df.v + j), vh0 = ld4_state<kStreamState>(df.vhat + j);
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        const uint16_t *srow = df.signs_prev + (int64_t)t * kThreads + tid;
        const int64_t sstride = (int64_t)n_tiles * kThreads;
        const bool first_tile = (t == b * tb.uniform_tiles);
        for (int c0 = 0; c0 < n; c0 += kScaleChunk) {
            const int cn = min(kScaleChunk, n - c0);
            __syncthreads();
            for (int u = tid; u < cn; u += kThreads) {          // one thread per worker: the scale of this tile's block
                const float s = fused_block_scale(df.partial_prev + (int64_t)(c0 + u) * tb.n_pieces, b, tb, n_tiles, d);
                s_lds[u] = s;
                if (first_tile && r == 0) df.scales_out[(int64_t)(c0 + u) * tb.n_blocks + b] = s;
            }
            __syncthreads();
            for (int u0 = 0; u0 < cn; u0 += kSignBatch) {
                uint32_t bits[kSignBatch];
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) bits[u] = (u0 + u < cn) ? (uint32_t)srow[(c0 + u0 + u) * sstride] : 0u;
#pragma unroll
                for (int u = 0; u < kSignBatch; ++u) {
                    if (u0 + u < cn) {
                        const float s = s_lds[u0 + u];
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[c] = fadd(acc[c], signed_scale(s, bits[u], r * 4 + c));
                    }
                }
            }
        }
        // padding coordinates take no gradient
        const float4 gbar = make_float4(j < d ? fdiv(acc[0], df.p.n_workers) : 0.f, j + 1 < d ? fdiv(acc[1], df.p.n_workers) : 0.f,
                                        j + 2 < d ? fdiv(acc[2], df.p.n_workers) : 0.f, j + 3 < d ? fdiv(acc[3], df.p.n_workers) : 0.f);
        float4 th = th0, mm = m0, vv = v0, vh = vh0;
        amsgrad_update4(th, mm, vv, vh, gbar, df.p);
        st4_state<kStreamState>(df.theta + j, th);
        st4_state<kStreamState>(df.m + j, mm);
        st4_state<kStreamState>(df.v + j, vv);
        st4_state<kStreamState>(df.vhat + j, vh);
        return;
    }

    // ---- the pass of worker i over tile t (one piece: the tile lies inside block b)
    const int i = blockIdx.y - 4;
    const G *grow = g + (int64_t)i * d;
    float *xrow = xs + (int64_t)i * ld;
    GradRaw<G> gv[4];
    float4 xv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        gv[r] = load_raw4<false>(grow, j, d);
        xv[r] = ld4_row(xrow + j, tb.stream_rows);
    }
    const float s_prev = kPending ? fused_block_scale(df.partial_prev + (int64_t)i * tb.n_pieces, b, tb, n_tiles, d) : 0.f;
    float x[4][4];
    uint32_t sign_bits = 0;
    double a64 = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        const float4 g4 = widen4(gv[r]);
        const float gg[4] = {g4.x, g4.y, g4.z, g4.w};
        const float xx[4] = {xv[r].x, xv[r].y, xv[r].z, xv[r].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float e = kPending ? deferred_sign_error(xx[c], s_prev) : xx[c];
            x[r][c] = (j + c < d) ? fadd(gg[c], e) : 0.f;
        }
        st4_stream(xrow + j, make_float4(x[r][0], x[r][1], x[r][2], x[r][3]));
#pragma unroll
        for (int c = 0; c < 4; ++c) sign_bits |= (__float_as_uint(x[r][c]) >> 31) << (r * 4 + c);
    }
    signs[((int64_t)i * n_tiles + t) * kThreads + tid] = (uint16_t)sign_bits;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) a64 += (double)fabsf(x[r][c]);
    const double S = block_sum(a64, scratch);
    if (tid == 0) partial[(int64_t)i * tb.n_pieces + t] = S;
}

// Wire form of one message: the n_scales scales (none where only the bits are wanted), then the sign bits: output word
// q holds the coordinates 32 q .. 32 q + 31, bit j % 32 for coordinate j (set = negative), zero past d.  Those 32
// coordinates are eight consecutive float4 of one row r of the tile, i.e. the r-th nibble of eight consecutive sign
// words, which one 16-byte load brings in.  A launch of a few microseconds, bound by latency: the scales ride in it, since
// a copy of their own took as long again.
__global__ __launch_bounds__(kThreads) void bs_pack_message(const float *__restrict__ scales, int32_t n_scales,
                                                            const uint16_t *__restrict__ words, int64_t d,
                                                            float *__restrict__ out_scales, uint32_t *__restrict__ out_bits)
{
    const int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (q < n_scales) out_scales[q] = scales[q];
    if (q * 32 >= d) return;
    const int64_t t = (q * 32) / kTile;
    const int vec0 = (int)((q * 32) % kTile) / 4;            // first of the eight float4
    const int r = vec0 / kThreads, tid0 = vec0 % kThreads;   // tid0: a multiple of 8
    const uint4 w = *reinterpret_cast<const uint4 *>(words + t * kThreads + tid0);
    const uint32_t pair[4] = {w.x, w.y, w.z, w.w};
    uint32_t bits = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        bits |= (((pair[u] >> (r * 4)) & 0xfu) | (((pair[u] >> (16 + r * 4)) & 0xfu) << 4)) << (8 * u);
    const int64_t left = d - q * 32;
    if (left < 32) bits &= (1u << left) - 1u;
    out_bits[q] = bits;
}

// e_i of one worker in its defined form, from the stored x and the pending scales.  out may be xrow itself
// (every thread reads its own element before it writes it).
template <bool kPending>
__global__ __launch_bounds__(kThreads) void bs_materialize_error(const float *xrow, int64_t d, BsTable tb,
                                                                 const float *__restrict__ sp, float *out)
{
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= d) return;
    float e = xrow[j];
    if (kPending) {
        const int t = (int)(j / kTile);
        int q = tb.tile_piece0[t];
        const int q1 = tb.tile_piece0[t + 1];
        while (q + 1 < q1 && j >= tb.piece_hi[q]) ++q;
        e = deferred_sign_error(e, sp[tb.piece_blk[q]]);
    }
    out[j] = e;
}

// CD-Adam, Algorithm 1, lines 10 and 12-16: gtilde += c with c = copysign(s[block], w) from the
// server's sign bits and scales, then the AMSGrad update with gtilde.  One workgroup per tile.
template <bool kStreamState>
__global__ __launch_bounds__(kThreads) void bs_apply(int64_t d, BsTable tb, const float *__restrict__ scales,
                                                     const uint16_t *__restrict__ signs, float *__restrict__ gtil,
                                                     float *__restrict__ theta, float *__restrict__ m,
                                                     float *__restrict__ v, float *__restrict__ vhat, AmsParams p)
{
    __shared__ uint16_t bound[kTile];                // piece ends of a tile where several blocks meet
    const int t = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)t * kTile;
    const uint32_t bits = signs[(int64_t)t * kThreads + tid];
    float4 gt[4], th[4], mm[4], vv[4], vh[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        gt[r] = ld4(gtil + j);
        th[r] = ld4_state<kStreamState>(theta + j);
        mm[r] = ld4_state<kStreamState>(m + j);
        vv[r] = ld4_state<kStreamState>(v + j);
        vh[r] = ld4_state<kStreamState>(vhat + j);
    }
    int p0, p1;
    if (tb.uniform_tiles > 0) {
        p0 = t;
        p1 = t + 1;
    } else {
        p0 = tb.tile_piece0[t];
        p1 = tb.tile_piece0[t + 1];
    }
    const bool single = (p1 - p0 == 1);
    const int P = p1 - p0;
    const int b0 = tb.uniform_tiles > 0 ? t / tb.uniform_tiles : tb.piece_blk[p0];   // block of the tile's first piece
    const float s_single = single ? scales[b0] : 0.f;
    if (!single) stage_piece_bounds(bound, p0, p1, tb, base);                         // uniform over the workgroup
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        const int l0 = 4 * (tid + kThreads * r);
        const float old[4] = {gt[r].x, gt[r].y, gt[r].z, gt[r].w};
        float nt[4];
        int q = single ? 0 : piece_index(bound, P, l0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float s = s_single;
            if (!single) {
                while (q + 1 < P && l0 + c >= (int)bound[q]) ++q;
                s = scales[b0 + q];
            }
            nt[c] = (j + c < d) ? fadd(old[c], signed_scale(s, bits, r * 4 + c)) : old[c];   // padding stays 0
        }
        const float4 g4 = make_float4(nt[0], nt[1], nt[2], nt[3]);
        amsgrad_update4(th[r], mm[r], vv[r], vh[r], g4, p);
        st4_state<kStreamState>(gtil + j, g4);
        st4_state<kStreamState>(theta + j, th[r]);
        st4_state<kStreamState>(m + j, mm[r]);
        st4_state<kStreamState>(v + j, vv[r]);
        st4_state<kStreamState>(vhat + j, vh[r]);
    }
}

// ghat_i of one worker in its defined form: the stored vector plus the pending c_i.  out may be xrow itself.
template <bool kPending>
__global__ __launch_bounds__(kThreads) void bs_materialize_markov(const float *xrow, int64_t d, BsTable tb,
                                                                  const float *__restrict__ sp,
                                                                  const uint16_t *__restrict__ signs_row, float *out)
{
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= d) return;
    float gh = xrow[j];
    if (kPending) {
        const int t = (int)(j / kTile);
        int q = tb.tile_piece0[t];
        const int q1 = tb.tile_piece0[t + 1];
        while (q + 1 < q1 && j >= tb.piece_hi[q]) ++q;
        // coordinate 4 * (tid + 256 * r) + c of the tile is bit r * 4 + c of the word of thread tid
        const int l = (int)(j - (int64_t)t * kTile);
        const int vec = l >> 2, c = l & 3;
        const uint32_t bits = signs_row[(int64_t)t * kThreads + (vec & (kThreads - 1))];
        gh = fadd(gh, signed_scale(sp[tb.piece_blk[q]], bits, (vec / kThreads) * 4 + c));
    }
    out[j] = gh;
}

}  // namespace cams
