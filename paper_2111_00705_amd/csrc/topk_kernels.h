// Top-k compression (Appendix A, "Top-k") with error feedback (Section 4), server average and
// AMSGrad update (Section 3).
//
// Selection is an exact radix select, not a sort.  Every element gets the composite key
//     comp = (magnitude_bits << IB) | (2^IB - 1 - index),     magnitude_bits = bits(x) & 0x7fffffff,
// IB = number of bits of d-1.  comp is unique per element and its descending order is
// "larger magnitude first, lower index first among equals", so Top-k is { comp >= Tc } where Tc is
// the k-th largest comp.  Tc is found digit by digit from the top.
//
// The error memory is kept in deferred form: after a step the library stores x_i = g_i + e_i and
// the worker's threshold Tc_i; e_i[j] = (comp(x_i[j], j) >= Tc_i) ? +0 : x_i[j] is formed on the fly
// when the next step (or a getter) reads x_i, so kept coordinates are never zeroed by scattered
// writes and one step needs a single pass over g and the stored vector.  Five launches per step,
// ordered only by kernel boundaries (no fences, no waiting inside a kernel):
//
//   tk_pass1    one workgroup per (tile, worker): streams g and the stored x once and writes the new
//               x; lists "candidates" - elements whose fine magnitude bin (top 17 bits, 0.2 % wide)
//               is >= the worker's guess, which is the previous step's threshold minus a little
//               slack - as (index, value) pairs, appended densely to one of 32 or 64 regions of the worker
//               (one atomic add per tile): straight from registers, or staged in LDS first (value and
//               place in the tile, 6 bytes), see kListStaged.
//               A workgroup per tile (instead of a loop over tiles) matters: on this chip a wave
//               that loops must wait for its stores before it can use its next loads.
//   tk_hist     histograms of the candidates: the fine bins of eight coarse bins (see window_start),
//               coarse bins (top 11 bits) outside; with fewer than k candidates (always on the first
//               step) the guess was too high: then the workgroups count the whole vector into a
//               full coarse histogram instead
//   tk_compact  coarse and fine bin of the k-th largest (every workgroup for itself); candidates in
//               that threshold bin are copied, as comp values, to dense pieces (one per wavefront);
//               after such a miss: the candidates are listed again from the stored x
//   tk_resolve  one workgroup per worker: the remaining digits of Tc over those pieces, and the
//               guess for the next step
//               (in place of the last three: tk_small_select, one workgroup per worker, see one_launch_select)
//   tk_final    per tile, all workers: candidates with comp >= Tc are the kept coordinates; their
//               values are added into an LDS copy of the tile in ascending worker order; then
//               gbar = acc / n and the AMSGrad update of the tile's theta, m, v, vhat
//
// Traffic per (worker, coordinate): 4 B g + 4 B stored x read + 4 B x written, plus the candidates
// (about 1.2 k per worker, 8 B each, written once, read three times).
//
// The candidate regions are bounded (see region_base): a region that fills up is detected, and the step then
// goes the way of a guess that was too high (whole-vector count, lists made anew) and, if the lists still do not
// fit, selects without lists inside tk_resolve (exact_select).  In vectors of at most 16 tiles, and in those whose lists one
// workgroup holds (one_launch_select), one kernel
// (tk_small_select) takes the place of tk_hist, tk_compact and tk_resolve, but for a first step beyond four tiles.
//
// Exact zeros under error feedback: when fewer than k coordinates are non-zero the k-th largest is a zero and
// zeros are selected by lower index.  They are never listed as candidates (millions of equal keys would be);
// tk_pass1 counts them per tile, and tk_resolve (or tk_small_select, but on short vectors) places the threshold among them from
// those counts (zero_tail_threshold).  The other methods list zeros like any other value.
//
// Rand-k (Appendix A, "Rand-k") runs through the same kernels: the 31 magnitude bits are replaced by a
// 31-bit pseudo-random score of (seed, step, worker, index), see SelKey; everything after the key -
// bins, digits, thresholds, the deferred error - is unchanged.
#pragma once
#include "device_utils.h"
#include "launch_rules.h"

namespace cams {

constexpr int kBins1 = 2048;      // coarse bin: top 11 of the 31 magnitude bits
constexpr int kShift1 = 20;
constexpr int kFineShift = 14;    // fine bin: top 17 bits; 64 fine bins per coarse bin
constexpr int kFinePerCoarse = 1 << (kShift1 - kFineShift);
constexpr int kWindowCoarse = 8;  // coarse bins whose fine bins are counted (see window_start): one octave of
                                  // magnitudes.  In the first steps of a run the threshold climbs by tens of fine
                                  // bins per step; beyond the window only the coarse bin is known and the threshold
                                  // bin holds 64 times the elements (with two coarse bins, n = 8, d = 110 M: steps
                                  // 1 to 6 spent 65-200 us in tk_resolve instead of 15)
constexpr int kFineWindow = kWindowCoarse * kFinePerCoarse;
constexpr int kDigitBits = 12;    // digits of the dense-array search
constexpr int kBins2 = 1 << kDigitBits;
constexpr int kFirstBits = 10;    // first digit below the prefix, counted by tk_compact while it copies: narrower,
                                  // since every one of its workgroups clears and flushes the bins
constexpr int kBinsFirst = 1 << kFirstBits;
constexpr int kPieceWords = kBinsFirst / 32;   // words of a dense piece's bitmap: which first digits occur in it
constexpr int kSub = kTile / 4;   // coordinates of a tile that one wavefront handles = capacity of its staged list
constexpr unsigned kStageBytes = 4 * kSub * (sizeof(float) + sizeof(uint16_t));   // staging lists of a workgroup of tk_pass1
constexpr int kMinSlices = 32;    // candidate regions per vector: a power of two in [kMinSlices, kMaxSlices]
                                  // (fewer for a vector of fewer tiles than that)
constexpr int kLongSlices = 64;   // from kLongTiles tiles on.  Fewer regions are fewer workgroups with histograms to flush, more
constexpr int kLongTiles = 512;   // are fewer atomic adds in a row on a cursor.  Step plus get_theta, 64 / 32 regions, us: error
                                  // feedback n = 8, d = 200 000 46.2 / 45.2, Rand-k n = 16, d = 1.2 M f16 93.0 / 91.8, CD-Adam n = 8,
                                  // d = 1 M 89.1 / 86.5; naive n = 8, d = 3 M bf16 79.7 / 80.4; d = 11 M and more equal
constexpr int kMaxSlices = 512;
constexpr int kCursorStride = 32; // words between two region cursors: a 128-byte line each.  The atomic adds of all XCDs on
                                  // one line are served one after the other, also where they go to different words (64
                                  // cursors on two lines: step plus get_theta, CD-Adam n = 8, d = 11.2 M bf16 387 us against
                                  // 377; naive n = 8, d = 3 M bf16 89 against 87)
constexpr int kMaxParts = 8;      // pieces a region is cut into for tk_hist / tk_compact, at most
constexpr int kResolveThreads = 1024;
constexpr uint32_t kNoGuess = 1u << 17;      // fine-bin guess that lists nothing (before the first step)
constexpr uint64_t kNoThreshold = ~0ull;     // Tc that keeps nothing (no pending selection)
constexpr uint32_t kMinSlack = 8, kMaxSlack = 512, kFirstSlack = 8;   // in fine bins (0.2 % each)
static_assert(kOneSelectSlack >= kMinSlack, "kMinSlack where one workgroup selects from several regions");
constexpr uint32_t kZeroTail = 2;            // value of TkWorker::whole
constexpr uint32_t kExact = 3;               // value of TkWorker::whole: exact_select has found Tc and listed the kept set


struct TkWorker {
    uint64_t tc;            // threshold composite of the last finished step (pending selection)
    uint32_t guess;         // pass 1 lists elements with fine bin >= guess
    uint32_t slack;         // fine bins kept between the threshold and the next guess
    // leading digits of the running step's Tc, written by tk_compact, read by tk_resolve
    uint32_t prefix;        // magnitude bits above pshift
    uint32_t pshift;        // kFineShift or kShift1: how many low magnitude bits are still open
    uint32_t rank;          // 1-based rank (from the top) of the k-th largest among elements with this prefix
    uint32_t whole;         // 1: all elements with this prefix are kept, Tc needs no further digit; kZeroTail: all
                            // candidates are kept and `rank` zeros besides (see zero_tail_threshold)
    uint32_t relisted;      // the guess was above the threshold: candidates are listed again
    uint32_t last_fine;     // fine bin of the previous threshold (to see how far thresholds move)
    uint32_t step_word;     // Rand-k: TkRand::step_now of the step that left tc - the draw the deferred error memory
                            // must be read with.  Kept in device memory, not in a kernel argument, so that a step
                            // replayed from a HIP graph (which repeats its draw) still reads its predecessor's.
    uint32_t overflow;      // tk_pass1 found a candidate region full: the lists are incomplete, tk_hist counts the
                            // whole vector instead (as after a guess that was too high)
    uint32_t overflow2;     // listing anew, tk_compact found a region full as well: tk_resolve selects without lists
                            // (exact_select)
    uint32_t pad_;
};
static_assert(sizeof(TkWorker) == 56, "TkWorker is copied between host and device as plain bytes");

// The record behind a handle's last holds no selection: its tc is the address of a word in host memory that says so when a guess has
// missed (0: no such word).  As an argument of tk_small_select the address cost it 0.2 to 0.4 of 8.5 us; here, read by the kernel's last
// instructions after a miss that is marked as rare, it costs steps that do not miss next to nothing (without / with it, us: CD-Adam
// n = 8, d = 300 000 56.0 / 56.2, error feedback d = 200 000 37.8 / 38.0, n = 16, d = 378 180 53.7 / 53.6; raised ahead of the listing
// 56.0 / 56.6, 37.8 / 37.9, 53.6 / 53.6).
inline TkWorker flag_record(const uint32_t *flag)
{
    TkWorker w{};
    w.tc = reinterpret_cast<uint64_t>(flag);
    return w;
}
__device__ __forceinline__ void raise_flag(const TkWorker &record)
{
    if (record.tc) __hip_atomic_store(reinterpret_cast<uint32_t *>(record.tc), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Rand-k: what the score of a coordinate depends on besides its index and the vector's number.
struct TkRand {
    uint32_t on;          // 0: Top-k (keys are magnitudes)
    uint32_t seed_hi;     // upper half of the 64-bit seed
    uint32_t step_now;    // mix32(lower half of the seed + draw * 0x9e3779b9) for the running step's draw (the draw of
                          // the step whose selection is still pending is TkWorker::step_word)
    uint32_t who0;        // number of vector 0 of this geometry: 0 for the workers, n for CD-Adam's server
    uint32_t min_slack;   // Rand-k: least slack of the guess, in fine bins (0: kMinSlack).  The k-th largest score
                          // of a fresh draw scatters by sqrt(k (1 - k/d)) / d of the key range around (1 - k/d).
};

struct TkGeom {
    int64_t d, ld;
    int32_t n, n_tiles;
    int32_t idx_bits;       // IB
    uint32_t k;
    int32_t slices;         // candidate regions per vector (see region_base)
    int32_t slice_tiles;    // tiles that append to one candidate region = ceil(n_tiles / slices)
    uint32_t region_cap;    // entries a candidate region holds (see region_base)
    int32_t parts;          // tk_hist / tk_compact: workgroups per region
    int32_t relist_wgs;     // workgroups per worker that tk_compact lists with after a miss (each loops over tiles)
    int32_t stream_rows;    // the stored rows are too large to stay cached between steps: tk_pass1 loads them as a stream
    int32_t xcd_chunk;      // tk_pass1: tile_of_block's chunk
    TkRand rand;
};

// The 31-bit key that orders the coordinates of one vector: the magnitude bits (Top-k), or the score
//     mix32(mix32(j + a) ^ b) >> 1,   a = mix32(step ^ seed_hi ^ who * 0x85ebca6b),  b = mix32(a + 0xc2b2ae35)
// (Rand-k), mix32 being the 32-bit finaliser of MurmurHash3.  For a fixed vector and step the score is a
// bijection of the index followed by a shift, so at most two coordinates share it.
struct SelKey {
    uint32_t on, a, b;
};
__device__ __forceinline__ uint32_t mix32(uint32_t h)
{
    h ^= h >> 16;
    h *= 0x85ebca6bu;
    h ^= h >> 13;
    h *= 0xc2b2ae35u;
    h ^= h >> 16;
    return h;
}
__device__ __forceinline__ SelKey sel_key_of(const TkRand &r, uint32_t per_step, int vec)
{
    SelKey s;
    s.on = r.on;
    s.a = mix32(per_step ^ r.seed_hi ^ ((r.who0 + (uint32_t)vec) * 0x85ebca6bu));
    s.b = mix32(s.a + 0xc2b2ae35u);
    return s;
}
__device__ __forceinline__ uint32_t sel_key(const SelKey &s, float x, uint32_t j)
{
    return s.on ? mix32(mix32(j + s.a) ^ s.b) >> 1 : mag_key(x);
}

__device__ __forceinline__ uint64_t composite(uint32_t key, uint32_t j, int idx_bits)
{
    const uint64_t inv = ((1ull << idx_bits) - 1ull) - (uint64_t)j;
    return ((uint64_t)key << idx_bits) | inv;
}

// Pending selection of the previous step in 32-bit form: the coordinate j with key
// `key` was kept iff  key > tkey  or  (key == tkey and j <= tj).
struct KeptTest {
    uint32_t tkey, tj;
};
__device__ __forceinline__ KeptTest kept_test(uint64_t tc, int idx_bits)
{
    const uint32_t imask = (uint32_t)((1ull << idx_bits) - 1ull);
    KeptTest k;
    k.tkey = (uint32_t)(tc >> idx_bits);            // kNoThreshold gives 0xffffffff: above every key
    k.tj = imask - ((uint32_t)tc & imask);
    return k;
}
__device__ __forceinline__ bool was_kept(const KeptTest &k, uint32_t key, uint32_t j)
{
    return key >= k.tkey && (key > k.tkey || j <= k.tj);
}

// The first digit below the prefix of Tc (kFirstBits bits): a function of comp that does not decrease, over the elements
// that carry the prefix.
// Where the prefix is a fine bin (kFineShift magnitude bits open) one bit of the digit is the top open bit, and half of the
// values that leaves go to the elements whose further open bits are all zero, by the top bits of their index; the others
// share the rest by magnitude.  16-bit gradients have no further bits: what ties there are told apart by their index in this
// digit already, where with the top kFirstBits open bits all of them carried the same one (tk_resolve, naive n = 8,
// d = 3 M bf16, 12.6 -> 8.3 us; step plus get_theta 73.8 -> 71.3, CD-Adam n = 8, d = 11.2 M bf16 342.5 -> 336, naive n = 16,
// d = 11 M f16 with 5 % kept 285 -> 279).  Elsewhere, and for scores (Rand-k), which have no ties, the digit is the top
// kFirstBits open bits.
struct FirstDigit {
    int idx_bits, s_lo;         // s_lo: comp bits below the digit, when it is a run of bits
    bool split;
};
constexpr uint32_t kTieBins = kBinsFirst / 4;      // per value of the top open bit
constexpr int kTieBits = kFirstBits - 2;
constexpr int kRestShift = kFineShift - 1 - kTieBits;      // magnitude bits below the digit of the others
static_assert(kRestShift >= 0, "magnitudes of a half in kTieBins bins");
static_assert(kShift1 - kFirstBits <= kFineShift, "a first digit below a coarse bin lies in one fine bin");
__device__ __forceinline__ FirstDigit first_digit(const TkGeom &ge, uint32_t pshift)
{
    return {ge.idx_bits, (int)pshift + ge.idx_bits - kFirstBits, pshift == (uint32_t)kFineShift && !ge.rand.on};   // pshift > kFirstBits
}
__device__ __forceinline__ uint32_t digit_of(const FirstDigit &f, uint64_t comp)
{
    if (!f.split) return (uint32_t)(comp >> f.s_lo) & (uint32_t)(kBinsFirst - 1);
    const uint32_t open = (uint32_t)(comp >> f.idx_bits) & ((1u << kFineShift) - 1u);
    const uint32_t half = open >> (kFineShift - 1), low = open & ((1u << (kFineShift - 1)) - 1u);
    const uint32_t inv = (uint32_t)comp & (uint32_t)((1ull << f.idx_bits) - 1ull);
    return half * 2u * kTieBins + (low == 0u ? inv >> (f.idx_bits - kTieBits) : kTieBins + (low >> kRestShift));
}
// The bits of comp, above the `open` lowest, that all elements with that digit under the prefix share; no element of a greater
// digit does.  (Ties share those of the smallest other magnitudes, which are greater: an element's rank from the top among those
// with its digit is its rank among those with these bits.)
struct DigitBits {
    uint64_t prefix;
    int open;
};
__device__ __forceinline__ DigitBits digit_bits(const FirstDigit &f, uint32_t prefix, uint32_t digit)
{
    if (!f.split) return {((uint64_t)prefix << kFirstBits) | digit, f.s_lo};
    const uint32_t half = digit / (2u * kTieBins), rest = digit % (2u * kTieBins);
    const uint64_t top = (uint64_t)prefix << 1 | half;
    if (rest < kTieBins) return {top << (kFineShift - 1 + kTieBits) | rest, f.idx_bits - kTieBits};
    return {top << kTieBits | (rest - kTieBins), f.idx_bits + kRestShift};
}
// The smallest comp of that digit under the prefix.
__device__ __forceinline__ uint64_t digit_edge(const FirstDigit &f, uint32_t prefix, uint32_t digit)
{
    const DigitBits b = digit_bits(f, prefix, digit);
    // the others' first digit begins above the ties
    const bool above_ties = f.split && digit % (2u * kTieBins) == kTieBins;
    return (b.prefix << b.open) + (above_ties ? 1ull << f.idx_bits : 0ull);
}

// Sums of the wavefronts of a workgroup of kWaves (a power of two up to 16) in part[]: the sum over those behind `wave`, uniform.
template <int kWaves>
__device__ __forceinline__ uint32_t waves_behind(const uint32_t *part, int wave)
{
    const int lane = threadIdx.x & 63;
    return scan_total(wave_scan(lane < kWaves && lane > wave ? part[lane & (kWaves - 1)] : 0u));
}

// The same over those before `wave`, of a workgroup of kResolveThreads.
__device__ __forceinline__ uint32_t waves_before(const uint32_t *part, int wave)
{
    const int lane = threadIdx.x & 63;
    return scan_total(wave_scan(lane < wave ? part[lane & (kResolveThreads / kWave - 1)] : 0u));
}

// Finds, in a histogram of kBins counters held in LDS by a workgroup of kResolveThreads, the bin
// of the element of 1-based rank `rank` counted from the top bin downwards, and leaves
// {bin, elements in higher bins, the bin's count} in res[0..2] for every thread (res[3] = 1 if
// found, which needs 1 <= rank <= total).  `part` holds one LDS counter per wavefront.  Bound by latency (wave_scan; tk_compact
// and tk_resolve together, us, with shuffles and the wavefronts' counters read one after the other / now: Rand-k n = 16, d = 1.2 M f16
// 11.1 / 9.8, naive n = 8, d = 3 M bf16 14.1 / 12.1).
template <int kBins>
__device__ __forceinline__ void find_rank_bin(const uint32_t *lh, uint32_t *part, uint32_t *res, uint32_t rank)
{
    constexpr int per = kBins / kResolveThreads;
    static_assert(per * kResolveThreads == kBins, "the same number of bins for every thread");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t own[per], mine = 0;
#pragma unroll
    for (int q = 0; q < per; ++q) {
        own[q] = lh[threadIdx.x * per + q];
        mine += own[q];
    }
    const uint32_t incl = wave_scan(mine), total = scan_total(incl);
    if (lane == 0) part[wave] = total;
    if (threadIdx.x == 0) res[3] = 0;
    __syncthreads();
    uint32_t above = waves_behind<kResolveThreads / kWave>(part, wave) + total - incl;
    if (above < rank && above + mine >= rank) {
        bool found = false;
#pragma unroll
        for (int q = per - 1; q >= 0; --q) {
            if (!found && above + own[q] >= rank) {
                res[0] = threadIdx.x * per + q;
                res[1] = above;
                res[2] = own[q];
                res[3] = 1;
                found = true;
            }
            above += own[q];
        }
    }
    __syncthreads();
}

// The same for a histogram of 8 * kThreads bins held in registers by a workgroup of kThreads: thread t owns the bins
// 8 t .. 8 t + 7.
__device__ __forceinline__ void find_rank_owned(const uint32_t (&own)[8], uint32_t *part, uint32_t *res, uint32_t rank)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) mine += own[q];
    const uint32_t incl = wave_scan(mine), total = scan_total(incl);
    if (lane == 0) part[wave] = total;
    __syncthreads();
    uint32_t above = waves_behind<kThreads / kWave>(part, wave) + total - incl;
    if (above < rank && above + mine >= rank) {
        bool found = false;
#pragma unroll
        for (int q = 7; q >= 0; --q) {
            if (!found && above + own[q] >= rank) {
                res[0] = threadIdx.x * 8 + q;
                res[1] = above;
                res[2] = own[q];
                found = true;
            }
            above += own[q];
        }
    }
    __syncthreads();
}

// Appends this wavefront's flagged lanes to a list: returns the slot of the calling lane (valid
// where flag is set) and advances count (uniform over the wavefront).
__device__ __forceinline__ uint32_t wave_append(bool flag, uint32_t &count)
{
    const uint64_t mask = __ballot(flag);
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t slot = count + __popcll(mask & ((1ull << lane) - 1ull));
    count += __popcll(mask);
    return slot;
}

// ---------------------------------------------------------------------------------------------
// Where candidates live.  Each worker owns ge.slices regions of ge.region_cap entries in the candidate array,
// one after the other; tile t appends to region t mod slices, so workgroups that run at the same time
// (neighbouring tiles) use different cursors, on different lines (kCursorStride).  Atomic adds on one cursor are served one
// after the other, on a busy chip at up to a microsecond each, so a single long vector (CD-Adam's server) takes more regions
// than each of many workers.  A tile takes its space with one atomic add
// on the region's cursor and records {offset from the worker's first region, counts of its four wavefronts,
// zeros} in the tile directory; inside the tile's space the candidates stand wavefront by wavefront.  The
// order of the tiles inside a region depends on timing; nothing downstream depends on it (comp values are
// unique, the selection is a set).  Appending densely matters: per-tile fixed slots made the same kernel
// 10 - 20 % slower (8-byte pieces scattered over gigabytes).
//
// A region holds a bounded number of entries (the host sizes a worker's regions for twice max(4 k, d / 64)
// candidates in all; 1.2 k are listed in steady state), not every coordinate of its tiles.  A tile that does not
// fit sets the worker's overflow flag and stores nothing: the worker's lists are then incomplete and the step
// goes on as after a guess that was too high - tk_hist counts the whole vector and tk_compact lists again with
// the coarse bin of the k-th largest; if that does not fit either (thousands of equal magnitudes: nothing
// narrower than the whole composite key separates them), tk_resolve selects without lists (exact_select).
__device__ __forceinline__ int64_t worker_base(const TkGeom &ge, int worker)
{
    return (int64_t)worker * ge.slices * ge.region_cap;
}
__device__ __forceinline__ int64_t region_base(const TkGeom &ge, int worker, int slice)
{
    return region_first(worker, ge.slices, slice, ge.region_cap);
}

// Takes `total` entries of region (i, t mod slices) for tile t and writes the tile's directory record; one
// thread calls this.  cnt: the candidates of the tile's four wavefronts (each below 2^16: a wavefront owns
// kSub = 1024 coordinates).  Returns the offset of the tile's space from the worker's first region, or
// kNoSpace when the region is full - the record then says that nothing is stored and *overflow_flag is set.
constexpr uint32_t kNoSpace = 0xffffffffu;
__device__ __forceinline__ uint32_t take_space(const uint32_t (&cnt)[4], uint32_t zeros, const TkGeom &ge, int i, int t,
                                               uint32_t *__restrict__ cursor, uint4 *__restrict__ tile_dir,
                                               uint32_t *overflow_flag)
{
    const uint32_t total = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    const int slice = t & (ge.slices - 1);
    uint32_t at = 0;
    if (total) {
        at = atomicAdd(cursor + (i * ge.slices + slice) * kCursorStride, total);
        if (at > ge.region_cap || total > ge.region_cap - at) {
            *overflow_flag = 1u;
            tile_dir[(int64_t)i * ge.n_tiles + t] = make_uint4(0u, 0u, 0u, zeros);
            return kNoSpace;
        }
    }
    at += (uint32_t)slice * ge.region_cap;
    tile_dir[(int64_t)i * ge.n_tiles + t] = make_uint4(at, cnt[0] | (cnt[1] << 16), cnt[2] | (cnt[3] << 16), zeros);
    return at;
}

// The space of one tile for a workgroup of four wavefronts that have counted their candidates (count, and zeros: the
// wavefront's count of exact zeros; the tile's sum goes into the directory record).  Leaves the four counts in
// sh[0 .. 3] and the offset (or kNoSpace) in sh[4], with a barrier after them.  sh: 9 LDS words.
__device__ __forceinline__ void take_tile_space(uint32_t count, uint32_t zeros, uint32_t *sh, const TkGeom &ge, int i,
                                                int t, uint32_t *__restrict__ cursor, uint4 *__restrict__ tile_dir,
                                                uint32_t *overflow_flag)
{
    const int tid = threadIdx.x;
    if ((tid & 63) == 0) {
        sh[tid >> 6] = count;
        sh[5 + (tid >> 6)] = zeros;
    }
    __syncthreads();
    if (tid == 0) {
        const uint32_t cnt[4] = {sh[0], sh[1], sh[2], sh[3]};
        sh[4] = take_space(cnt, sh[5] + sh[6] + sh[7] + sh[8], ge, i, t, cursor, tile_dir, overflow_flag);
    }
    __syncthreads();
}

// A wavefront's staged candidates, in the passes that stage them (kListStaged): the value and the
// coordinate's place inside the tile, 6 bytes per entry instead of the 8 of an (index, value) pair.  With room for every
// coordinate of the wavefront (so the list cannot overflow) a workgroup's four lists take 24 KB, and six workgroups fit a
// compute unit where 32 KB allowed four: CD-Adam's passes, which only read, run 3-5 % faster with the additional loads in
// flight.
struct Stage {
    float *val;          // [kSub]
    uint16_t *at;        // [kSub] index - first index of the tile
};

// Stages one element of the vector that is compressed as a candidate if its fine bin reaches the guess.
// base: first index of the tile.
// kSkipZeros (error feedback with magnitude keys): exact zeros are never listed but counted (zeros, uniform
// over the wavefront) - when fewer than k coordinates are non-zero the threshold lies among the zeros, which
// are ordered by index alone, and is placed from these counts instead (see zero_tail_threshold).
template <bool kSkipZeros>
__device__ __forceinline__ void consider(float x, uint32_t j, uint32_t base, bool valid, uint32_t guess, const SelKey &sk,
                                         const Stage &stage, uint32_t &count, uint32_t &zeros)
{
    bool hit = valid && (sel_key(sk, x, j) >> kFineShift) >= guess;
    if (kSkipZeros && !sk.on) {
        const bool zero = valid && mag_key(x) == 0u;
        zeros += (uint32_t)__popcll(__ballot(zero));
        hit = hit && !zero;
    }
    const uint32_t slot = wave_append(hit, count);
    if (hit) {
        stage.val[slot] = x;
        stage.at[slot] = (uint16_t)(j - base);
    }
}

// One tile of one worker.  kFull: the whole tile lies below d.  Candidates are staged in LDS (one
// list per wavefront, which owns kSub coordinates of the tile, so it cannot overflow).
// Modes: kPassEf  error feedback: x = g + e, written back over the stored vector;
//        kPassCd  CD-Adam worker (Algorithm 1, line 5): u = g - ghat_i, nothing written back (ghat_i
//                 changes only where c_i is not zero; tk_merge does that);
//        kPassNaive  naive compression (Section 4): x = g, the stored rows are not touched.
enum { kPassEf = 0, kPassCd = 1, kPassNaive = 3 };

// The gradients and the stored values of this thread's coordinates, base + 4 (tid + 256 r) + c.  kFull: the whole tile lies
// below d.
template <bool kFull, int kMode, typename G>
__device__ __forceinline__ void load_pass_tile(GradRaw<G> (&gv)[4], float4 (&xv)[4], const G *__restrict__ grow,
                                               const float *__restrict__ xrow, uint32_t base, uint32_t d, int stream_rows)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t j = base + 4 * (threadIdx.x + kThreads * r);
        gv[r] = load_raw4<kFull>(grow, j, d);
        xv[r] = kMode == kPassNaive ? make_float4(0.f, 0.f, 0.f, 0.f) : ld4_row(xrow + j, stream_rows);
    }
}

// The coordinates j .. j + 3 of the vector that is compressed; under error feedback they are stored as well.
template <bool kFull, int kMode>
__device__ __forceinline__ void form_coordinates(float (&x)[4], const float4 &g, const float4 &old, uint32_t j, uint32_t d,
                                                 const KeptTest &kt, const SelKey &sk_prev, float *xrow)
{
    const float gg[4] = {g.x, g.y, g.z, g.w};
    const float xo[4] = {old.x, old.y, old.z, old.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (kMode == kPassNaive) {
            x[c] = (kFull || j + c < d) ? gg[c] : 0.f;
        } else if (kMode != kPassEf) {
            x[c] = (kFull || j + c < d) ? fsub(gg[c], xo[c]) : 0.f;
        } else {
            // e = x_old - C(x_old): +0 where the previous step kept the coordinate
            const float e = was_kept(kt, sel_key(sk_prev, xo[c], j + c), j + c) ? 0.f : xo[c];
            x[c] = (kFull || j + c < d) ? fadd(gg[c], e) : 0.f;
        }
    }
    if (kMode == kPassEf) st4_stream(xrow + j, make_float4(x[0], x[1], x[2], x[3]));
}

template <bool kFull, int kMode, typename G>
__device__ __forceinline__ uint32_t pass1_tile(const G *__restrict__ grow, float *__restrict__ xrow,
                                               uint32_t base, uint32_t d, const KeptTest &kt, uint32_t guess,
                                               const SelKey &sk, const SelKey &sk_prev, const Stage &stage,
                                               int stream_rows, uint32_t &zeros)
{
    const int tid = threadIdx.x;
    GradRaw<G> gv[4];
    float4 xv[4];
    load_pass_tile<kFull, kMode>(gv, xv, grow, xrow, base, d, stream_rows);
    uint32_t count = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t j = base + 4 * (tid + kThreads * r);
        float x[4];
        form_coordinates<kFull, kMode>(x, widen4(gv[r]), xv[r], j, d, kt, sk_prev, xrow);
#pragma unroll
        for (int c = 0; c < 4; ++c)
            consider<kMode == kPassEf>(x[c], j + c, base, kFull || j + c < d, guess, sk, stage, count, zeros);
    }
    return count;
}

// End of a tile whose candidates are staged.  No workgroup barrier: a wavefront that is done registers itself, and
// whichever of the four comes last does the rest for the whole tile - takes the tile's space in its
// region (one atomic add), writes the directory record and copies all staged candidates.  The other
// three leave at once instead of waiting for the atomic.
// sh: 9 LDS words, sh[4] zeroed (with a barrier after it) before the first wavefront can get here.
// zeros: this wavefront's count of exact zeros; the tile's sum goes into the directory record's last word.
__device__ __forceinline__ void finish_tile(const float (*stage_val)[kSub], const uint16_t (*stage_at)[kSub], uint32_t *sh,
                                            uint32_t count, uint32_t zeros,
                                            const TkGeom &ge, int i, int t, uint2 *__restrict__ cand,
                                            uint32_t *__restrict__ cursor, uint4 *__restrict__ tile_dir,
                                            uint32_t *overflow_flag)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // this wavefront's staged candidates are complete before it registers
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    uint32_t arrived = 0;
    if (lane == 0) {
        sh[wave] = count;
        sh[5 + wave] = zeros;
        arrived = __hip_atomic_fetch_add(&sh[4], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    arrived = __builtin_amdgcn_readfirstlane(arrived);
    if (arrived != 3) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");

    const uint32_t cnt[4] = {sh[0], sh[1], sh[2], sh[3]};
    uint32_t at = 0;
    if (lane == 0) at = take_space(cnt, sh[5] + sh[6] + sh[7] + sh[8], ge, i, t, cursor, tile_dir, overflow_flag);
    at = __builtin_amdgcn_readfirstlane(at);
    if (at == kNoSpace) return;
    uint2 *dst = cand + worker_base(ge, i) + at;
    const uint32_t base = (uint32_t)t * kTile;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        for (uint32_t q = lane; q < cnt[w]; q += kWave)
            dst[q] = make_uint2(base + stage_at[w][q], __float_as_uint(stage_val[w][q]));
        dst += cnt[w];
    }
}

// How tk_pass1 lists.  Staged: in LDS, and the last wavefront of a workgroup to finish copies all lists out alone.  Or straight from
// its registers: each wavefront counts its candidates, the workgroup takes the tile's space, and each wavefront writes its own, slot
// by slot of the wavefront or thread by thread with few instructions (list_registers).  A store then carries one or two candidates
// instead of a run of them, which costs nothing until they are many, and no LDS is held.  Step plus get_theta, us, staged / slot by
// slot: error feedback fp32 n = 16, d = 11.2 M 488 / 475, n = 8, d = 25 M 628 / 606, d = 110 M 2433 / 2418; naive compression (held at
// 64 registers: eight workgroups per unit where the lists allowed six) n = 8, d = 3 M bf16 83 / 80, n = 4, d = 60 M bf16 613 / 574,
// Rand-k n = 16, d = 6 M fp32 173 / 164 (Rand-k spilled one or two registers for that, and gained by it on 16 bits all the same:
// n = 16, d = 11.2 M f16 300 without the bound, 294 with it, fp32 266 / 266).  Staged / thread by thread: error feedback on 16 bits
// Rand-k n = 16, d = 1.2 M f16 80.4 / 79.6, Top-k bf16 80.1 / 79.4, n = 8, d = 300 000 f16 44.8 / 43.9, n = 4, d = 65 536 29.4 / 28.5,
// n = 8, d = 4 M 115.8 / 114.4, but n = 16, d = 11.2 M 398.5 / 399.1, n = 8, d = 60 M 1171 / 1202; CD-Adam n = 8, d = 20 000
// 41.0 / 40.1, but d = 2 M 103.4 / 106.6, d = 11.2 M bf16 335 / 345, n = 16 502 / 517.  The host's list_mode draws the lines.
enum { kListStaged = 0, kListSlots = 1, kListThreads = 2 };

// What the listing pass knows at compile time about the keys: magnitudes (Top-k), scores (Rand-k), or nothing.  Without
// a branch per element: step plus get_theta, us, n = 4, d = 65 536 33.5 / 32.7, n = 8, d = 2 M 89.3 / 87.9, n = 16, d = 11.2 M
// 462 / 459, Rand-k n = 16, d = 1.2 M f16 92.5 / 90.9, naive n = 8, d = 3 M bf16 79.2 / 77.8.  The long rows of error feedback on
// 32-bit gradients (tk_long_rows) keep the branch, as they want fewer workgroups per unit.  The pass alone, with / without the
// branch, mean and range over eight shapes of 70 M to 200 M coordinates and 2 to 16 workers: Top-k with k = 0.03 % to 0.4 % 1.4 %
// faster with it (4 % slower to 7 % faster), with 1 % equal (-2 to 1.4 %), Rand-k 0.1 % 2.6 % faster (-1.3 to 5 %), 1 % 1.7 % slower
// (-4.5 to 0.5 %); n = 8, d = 110 M, k = 0.1 % 1652 / 1677 us.  Five shapes of 11 M to 55 M, Top-k: 0.2 % slower (-1.9 to 1.5 %).
enum { kKeyMagnitude = 0, kKeyScore = 1, kKeyEither = 2 };

// Lists the candidates among this thread's 16 values of tile t straight from the registers (x[r][c]: coordinate
// base + 4 (tid + 256 r) + c), thread by thread.  kSkipZeros: see consider.  All threads of the workgroup call this.
// A value takes a subtraction, whose top bit says that its key lies below the guess, and a shift of that bit into a mask; one scan
// places a thread's candidates, which follow one another in the list.  Step plus get_theta, us, slot by slot / thread by thread:
// naive Rand-k n = 8, d = 3 M bf16 74.4 / 72.0, Top-k 68.4 / 68.2, d = 100 M 1110 / 1095, error
// feedback n = 4, d = 65 536 29.3 / 28.7, n = 8, d = 300 000 44.6 / 43.8, d = 2 M 83.2 / 81.8, Rand-k n = 16, d = 1.2 M 85.0 / 83.9; long rows
// under error feedback lose: n = 16, d = 11.2 M 455.1 / 457.2, n = 8, d = 25 M 587 / 592, d = 110 M 2374 / 2416.
template <bool kFull, bool kSkipZeros>
__device__ __forceinline__ void list_registers(const float (&x)[4][4], uint32_t base, uint32_t d, uint32_t guess, const SelKey &sk,
                                               uint32_t *sh, const TkGeom &ge, int i, int t, uint2 *__restrict__ cand,
                                               uint32_t *__restrict__ cursor, uint4 *__restrict__ tile_dir,
                                               uint32_t *overflow_flag)
{
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t first = guess << kFineShift;      // the smallest key that is listed; kNoGuess gives 2^31, above every key
    uint32_t below = 0, zero = 0;                    // bit 15 - (4 r + c)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t j = base + 4 * (tid + kThreads * r);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool valid = kFull || j + c < d;
            const uint32_t under = sel_key(sk, x[r][c], j + c) - first;
            below = __builtin_amdgcn_alignbit(below, valid ? under : ~0u, 31);
            if (kSkipZeros && !sk.on) zero = __builtin_amdgcn_alignbit(zero, valid ? mag_key(x[r][c]) - 1u : 0u, 31);
        }
    }
    const uint32_t hits = ~(below | zero) & 0xffffu;
    // this thread's counts and the wavefront's, zeros in the upper half (a wavefront owns 1024 coordinates)
    const uint32_t mine = __popc(hits) | (kSkipZeros ? (uint32_t)__popc(zero) << 16 : 0u);
    const uint32_t incl = wave_scan(mine), both = scan_total(incl);
    take_tile_space(both & 0xffffu, both >> 16, sh, ge, i, t, cursor, tile_dir, overflow_flag);
    const uint32_t space = sh[4];
    if (space == kNoSpace) return;
    // the region in 64 bits, uniform and known before the tile's space is; the lanes' places inside it in 32 (a chain of the space's
    // offset to a scalar register and a 64-bit sum of it: naive n = 8, d = 3 M bf16 67.4 us, this 67.1)
    const int slice = t & (ge.slices - 1);
    uint2 *dst = cand + region_base(ge, i, slice);
    uint32_t at = space - (uint32_t)slice * ge.region_cap + (wave > 0 ? sh[0] : 0u) + (wave > 1 ? sh[1] : 0u) + (wave > 2 ? sh[2] : 0u) +
                  ((incl - mine) & 0xffffu);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (hits & (0x8000u >> (r * 4 + c)))
                *at_offset(dst, at++) = make_uint2(base + 4 * (tid + kThreads * r) + c, __float_as_uint(x[r][c]));
}

// A tile of the listing pass listed straight from the registers, thread by thread (list_registers) or slot by slot: a ballot and a
// prefix for each of a wavefront's 16 slots, beside the row's stores.
template <bool kFull, int kMode, int kList, typename G>
__device__ __forceinline__ void pass1_direct(const G *__restrict__ grow, float *__restrict__ xrow, uint32_t base, uint32_t d,
                                             const KeptTest &kt, uint32_t guess, const SelKey &sk, const SelKey &sk_prev,
                                             int stream_rows, uint32_t *sh, const TkGeom &ge, int i, int t,
                                             uint2 *__restrict__ cand, uint32_t *__restrict__ cursor,
                                             uint4 *__restrict__ tile_dir, uint32_t *overflow_flag)
{
    const int tid = threadIdx.x, wave = tid >> 6;
    GradRaw<G> gv[4];
    float4 xv[4];
    load_pass_tile<kFull, kMode>(gv, xv, grow, xrow, base, d, stream_rows);
    float x[4][4];
    uint32_t count = 0, zeros = 0, hits = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t j = base + 4 * (tid + kThreads * r);
        form_coordinates<kFull, kMode>(x[r], widen4(gv[r]), xv[r], j, d, kt, sk_prev, xrow);
        if constexpr (kList == kListSlots) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bool valid = kFull || j + c < d;
                bool hit = valid && (sel_key(sk, x[r][c], j + c) >> kFineShift) >= guess;
                if (kMode == kPassEf && !sk.on) {
                    const bool zero = valid && mag_key(x[r][c]) == 0u;
                    zeros += (uint32_t)__popcll(__ballot(zero));
                    hit = hit && !zero;
                }
                count += (uint32_t)__popcll(__ballot(hit));
                hits |= (hit ? 1u : 0u) << (r * 4 + c);
            }
        }
    }
    if constexpr (kList != kListSlots) {
        list_registers<kFull, kMode == kPassEf>(x, base, d, guess, sk, sh, ge, i, t, cand, cursor, tile_dir, overflow_flag);
    } else {
        take_tile_space(count, zeros, sh, ge, i, t, cursor, tile_dir, overflow_flag);
        uint32_t at = sh[4];
        if (at == kNoSpace) return;
        for (int w = 0; w < wave; ++w) at += sh[w];
        uint2 *dst = cand + worker_base(ge, i);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bool hit = (hits >> (r * 4 + c)) & 1u;
                const uint32_t slot = wave_append(hit, at);
                if (hit) dst[slot] = make_uint2(base + 4 * (tid + kThreads * r) + c, __float_as_uint(x[r][c]));
            }
    }
}

// G: element type of g - float, or uint16_t (bfloat16 bits) for gradients handed over as bfloat16.
template <int kMode, int kKey, int kList, typename G>
__global__ __launch_bounds__(kThreads, kMode == kPassNaive ? 8 : 1) void tk_pass1(const G *__restrict__ g, float *__restrict__ xs, TkGeom ge,
                                                     TkWorker *ws, uint2 *__restrict__ cand,
                                                     uint32_t *__restrict__ cursor, uint4 *__restrict__ tile_dir)
{
    constexpr bool kDirect = kList != kListStaged;   // the lists are not used then, and take no LDS
    __shared__ float stage_val[kDirect ? 1 : 4][kSub];
    __shared__ uint16_t stage_at[kDirect ? 1 : 4][kSub];
    __shared__ uint32_t sh[9];
    const int t = tile_of_block(blockIdx.x, ge.xcd_chunk);
    if (t >= ge.n_tiles) return;
    const int i = blockIdx.y;
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const uint32_t guess = ws[i].guess;
    const KeptTest kt = kept_test(ws[i].tc, ge.idx_bits);
    SelKey sk = sel_key_of(ge.rand, ge.rand.step_now, i);
    SelKey sk_prev = sel_key_of(ge.rand, ws[i].step_word, i);
    if constexpr (kKey != kKeyEither) sk.on = sk_prev.on = kKey == kKeyScore ? 1u : 0u;
    const uint32_t d = (uint32_t)ge.d;
    const uint32_t base = (uint32_t)t * kTile;
    const G *grow = g + (int64_t)i * ge.d;
    float *xrow = xs + (int64_t)i * ge.ld;
    if constexpr (kDirect) {
        if (base + kTile <= d)
            pass1_direct<true, kMode, kList, G>(grow, xrow, base, d, kt, guess, sk, sk_prev, ge.stream_rows, sh, ge, i, t, cand,
                                         cursor, tile_dir, &ws[i].overflow);
        else
            pass1_direct<false, kMode, kList, G>(grow, xrow, base, d, kt, guess, sk, sk_prev, ge.stream_rows, sh, ge, i, t, cand,
                                          cursor, tile_dir, &ws[i].overflow);
    } else {
        if (tid == 0) sh[4] = 0;
        __syncthreads();
        uint32_t count, zeros = 0;
        const Stage stage{stage_val[wave], stage_at[wave]};
        if (base + kTile <= d)
            count = pass1_tile<true, kMode, G>(grow, xrow, base, d, kt, guess, sk, sk_prev, stage, ge.stream_rows, zeros);
        else
            count = pass1_tile<false, kMode, G>(grow, xrow, base, d, kt, guess, sk, sk_prev, stage, ge.stream_rows, zeros);
        finish_tile(stage_val, stage_at, sh, count, zeros, ge, i, t, cand, cursor, tile_dir, &ws[i].overflow);
    }
}

// ---------------------------------------------------------------------------------------------
// The kept values of a tile, summed over the workers, and the AMSGrad update of the tile (tk_final's work).
//
// A coordinate of a tile belongs to one wavefront - the same one in tk_pass1, tk_compact's listing and here -
// and a tile's candidates are stored wavefront by wavefront, so each wavefront can sum the kept values
// of its own coordinates without looking at the others: no workgroup barrier, and the ascending worker
// order of the sum is just the order of its own instructions (within one worker the coordinates of
// the kept candidates are distinct).
constexpr int kFinBatch = 8;   // workers whose candidates a wavefront has in flight at a time

// Adds, for the calling wavefront's coordinates of tile t, the kept values (comp >= Tc_i) of all
// workers into acc (LDS, kTile floats, zeroed by the caller for these coordinates) in ascending
// worker order.  ws: the records that hold the selection's thresholds (and, for Rand-k, the draw they were made
// with).  kScatter (CD-Adam, Algorithm 1, line 6): the kept value u = c_i[j] is also added to
// ghat_i[j] in `rows` ([n][ld]); the old values are fetched for a whole batch before they are used.
// wave: the wavefront of the listing pass whose list is read.
template <bool kScatter>
__device__ __forceinline__ void sum_kept_tile(float *acc, const TkGeom &ge, const TkWorker *__restrict__ ws,
                                              const uint2 *__restrict__ cand, const uint4 *__restrict__ tile_dir,
                                              int t, float *__restrict__ rows, int wave)
{
    const uint32_t base = (uint32_t)t * kTile;
    const int lane = threadIdx.x & 63;
    for (int w0 = 0; w0 < ge.n; w0 += kWave) {
        const int nw = min(kWave, ge.n - w0);
        // lane l: where worker w0 + l keeps this wavefront's candidates of the tile, and its threshold
        uint32_t my_start = 0, my_count = 0;
        uint64_t my_tc = kNoThreshold;
        SelKey my_sk = {0u, 0u, 0u};
        if (lane < nw) {
            const uint4 rec = tile_dir[(int64_t)(w0 + lane) * ge.n_tiles + t];
            const uint32_t c[4] = {rec.y & 0xffffu, rec.y >> 16, rec.z & 0xffffu, rec.z >> 16};
            my_start = rec.x;
            for (int q = 0; q < wave; ++q) my_start += c[q];
            my_count = c[wave];
            my_tc = ws[w0 + lane].tc;
            my_sk = sel_key_of(ge.rand, ws[w0 + lane].step_word, w0 + lane);
        }
        for (int wb = 0; wb < nw; wb += kFinBatch) {
            uint2 e[kFinBatch];
            uint32_t cnt[kFinBatch];
            bool keep[kFinBatch];
            float old[kFinBatch];
#pragma unroll
            for (int u = 0; u < kFinBatch; ++u) {
                const int w = min(wb + u, nw - 1);           // clamped: the copies past nw are not used
                cnt[u] = wb + u < nw ? (uint32_t)__shfl((int)my_count, w, kWave) : 0u;
                const uint32_t start = (uint32_t)__shfl((int)my_start, w, kWave);
                // no branch around the load (lanes past the list read the worker's first entry): in one, the compiler waits for
                // each load before the next is issued
                e[u] = cand[worker_base(ge, w0 + w) + ((uint32_t)lane < cnt[u] ? start + lane : 0u)];
            }
#pragma unroll
            for (int u = 0; u < kFinBatch; ++u) {
                const int w = min(wb + u, nw - 1);
                const uint32_t tc_lo = (uint32_t)__shfl((int)(uint32_t)my_tc, w, kWave);
                const uint32_t tc_hi = (uint32_t)__shfl((int)(uint32_t)(my_tc >> 32), w, kWave);
                const uint64_t tc = ((uint64_t)tc_hi << 32) | tc_lo;
                SelKey sk = {0u, 0u, 0u};
                if (ge.rand.on) sk = {1u, (uint32_t)__shfl((int)my_sk.a, w, kWave), (uint32_t)__shfl((int)my_sk.b, w, kWave)};
                keep[u] = (uint32_t)lane < cnt[u] &&
                          composite(sel_key(sk, __uint_as_float(e[u].y), e[u].x), e[u].x, ge.idx_bits) >= tc;
                old[u] = 0.f;
                if (kScatter && keep[u]) old[u] = rows[(int64_t)(w0 + w) * ge.ld + e[u].x];
            }
#pragma unroll
            for (int u = 0; u < kFinBatch; ++u) {
                const int w = min(wb + u, nw - 1);
                if (keep[u]) {
                    const float x = __uint_as_float(e[u].y);
                    const uint32_t l = e[u].x - base;
                    acc[l] = fadd(acc[l], x);
                    // stored as a stream: the row is not read again before the next step (step plus get_theta, us, ordinary store /
                    // this: CD-Adam n = 8, d = 11.2 M bf16 336.0 / 330.8, n = 16 fp32 501.5 / 493.8, Rand-k n = 8, d = 25 M 686 / 676, Top-k
                    // 0.1 % of d = 60 M 1152 / 1154; loaded as a stream as well 343.5, 511, 691, 1158)
                    if (kScatter)
                        __builtin_nontemporal_store(fadd(old[u], x), rows + (int64_t)(w0 + w) * ge.ld + e[u].x);
                }
                if (cnt[u] > (uint32_t)kWave) {
                    // more than 64 candidates of this worker in the wavefront's quarter of the tile (rare)
                    const uint32_t tc_lo = (uint32_t)__shfl((int)(uint32_t)my_tc, w, kWave);
                    const uint32_t tc_hi = (uint32_t)__shfl((int)(uint32_t)(my_tc >> 32), w, kWave);
                    const uint64_t tc = ((uint64_t)tc_hi << 32) | tc_lo;
                    const uint32_t start = (uint32_t)__shfl((int)my_start, w, kWave);
                    const SelKey sk = {ge.rand.on, (uint32_t)__shfl((int)my_sk.a, w, kWave),
                                       (uint32_t)__shfl((int)my_sk.b, w, kWave)};
                    const uint2 *src = cand + worker_base(ge, w0 + w) + start;
                    for (uint32_t q = kWave + lane; q < cnt[u]; q += kWave) {
                        const uint2 c = src[q];
                        const float x = __uint_as_float(c.y);
                        if (composite(sel_key(sk, x, c.x), c.x, ge.idx_bits) >= tc) {
                            const uint32_t l = c.x - base;
                            acc[l] = fadd(acc[l], x);
                            if (kScatter) {
                                float *gh = rows + (int64_t)(w0 + w) * ge.ld + c.x;
                                *gh = fadd(*gh, x);
                            }
                        }
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // next worker's adds come after these
            }
        }
    }
}

// Server average and AMSGrad update, one workgroup per tile.
template <bool kStreamState>
__global__ __launch_bounds__(kThreads) void tk_final(TkGeom ge, const TkWorker *__restrict__ ws,
                                                     const uint2 *__restrict__ cand,
                                                     const uint4 *__restrict__ tile_dir,
                                                     float *__restrict__ theta, float *__restrict__ m,
                                                     float *__restrict__ v, float *__restrict__ vhat, AmsParams p)
{
    __shared__ float acc[kTile];
    const int t = blockIdx.x;
    const int64_t base = (int64_t)t * kTile;
    const int tid = threadIdx.x;

#pragma unroll
    for (int r = 0; r < 4; ++r) st4(acc + 4 * (tid + kThreads * r), make_float4(0.f, 0.f, 0.f, 0.f));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    sum_kept_tile<false>(acc, ge, ws, cand, tile_dir, t, nullptr, tid >> 6);

    // the state is loaded only now: fewer live registers above (more workgroups per compute unit),
    // which measured faster than loading it first
    float4 th[4], mm[4], vv[4], vh[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int64_t j = base + 4 * (tid + kThreads * r);
        th[r] = ld4_state<kStreamState>(theta + j);
        mm[r] = ld4_state<kStreamState>(m + j);
        vv[r] = ld4_state<kStreamState>(v + j);
        vh[r] = ld4_state<kStreamState>(vhat + j);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = 4 * (tid + kThreads * r);
        const int64_t j = base + l;
        const float4 a = ld4(acc + l);
        const float4 gbar = make_float4(fdiv(a.x, p.n_workers), fdiv(a.y, p.n_workers), fdiv(a.z, p.n_workers),
                                        fdiv(a.w, p.n_workers));
        const float4 vh0 = vh[r];
        amsgrad_update4(th[r], mm[r], vv[r], vh[r], gbar, p);
        st4_state<kStreamState>(theta + j, th[r]);
        st4_state<kStreamState>(m + j, mm[r]);
        st4_state<kStreamState>(v + j, vv[r]);
        // with a sparse average vhat = max(vhat, v) moves at few coordinates (v only decays elsewhere)
        st4_if_changed<kStreamState>(vhat + j, vh[r], vh0);
    }
}

// The same with a quarter of a tile per workgroup, for vectors that leave the chip idle otherwise (see quarter_final): quarter
// w holds the coordinates of the listing pass's wavefront w, and wavefront r here updates row r of them (one float4 per lane,
// the state loaded before anything else).
// Bound by a chain of latencies: the records of all workers, then the candidates, are each loaded at once.  The candidates
// are dealt out to the 256 threads together, since a worker's list holds a dozen of them in a quarter; the kept values of
// kBatch workers at a time then go to a row of LDS each, with a bit per coordinate, and every thread adds its own
// coordinates in ascending worker order.  A wavefront that went through the lists
// worker by worker, eight workers' candidates in flight, each of the four for its own row, took (step plus get_theta, us, that / this)
// Rand-k n = 16, d = 1.2 M f16 89.8 / 80.9, d = 300 000 with 20 % kept 80.6 / 66.5, n = 32, d = 21 000 f16 44.9 / 37.0, Top-k n = 16,
// d = 1.2 M 91.0 / 86.9, n = 48, d = 200 000 with 5 % kept 93.2 / 81.4, n = 20, d = 600 000 with 5 % kept bf16 87.6 / 74.2, n = 2,
// d = 1.3 M 52.5 / 51.6, n = 4, d = 65 536 33.0 / 32.8 (the whole step's gain where other kernels changed as well).  The bits are cleared
// before the first barrier and the search for an entry's worker takes as many steps as n or the batch needs: with six steps
// for any n and a barrier more, the smallest vectors lost (n = 4, d = 730 bf16 27.6 -> 27.9, now 27.7; naive d = 994 26.1 -> 26.3,
// now 26.1; n = 48 above 84.6, 20 % kept 69.1).
constexpr int kShortHeld = 2;         // candidates a thread holds from the start
template <bool kStreamState, int kBatch>   // kBatch: workers whose kept values are in LDS at a time
__global__ __launch_bounds__(kThreads) void tk_final_short(TkGeom ge, const TkWorker *__restrict__ ws,
                                                     const uint2 *__restrict__ cand,
                                                     const uint4 *__restrict__ tile_dir,
                                                     float *__restrict__ theta, float *__restrict__ m,
                                                     float *__restrict__ v, float *__restrict__ vhat, AmsParams p)
{
    __shared__ float val[kBatch][4 * kThreads];
    __shared__ uint32_t kept[kBatch][kWave];     // a word per thread of the listing pass: bit 4 r + c for row r, component c
    __shared__ uint32_t start[kShortFinalWorkers], upto[kShortFinalWorkers + 1], key_a[kShortFinalWorkers], key_b[kShortFinalWorkers];
    __shared__ uint64_t tc[kShortFinalWorkers];
    static_assert(kShortFinalWorkers <= kWave, "a worker per lane");
    const int t = blockIdx.x >> 2, w = blockIdx.x & 3;
    const int tid = threadIdx.x;
    const int lane = tid & 63, r = tid >> 6;
    const uint32_t base = (uint32_t)t * kTile;
    const int64_t j = (int64_t)base + 1024 * r + 256 * w + 4 * lane;
    float4 th = ld4_state<kStreamState>(theta + j), mm = ld4_state<kStreamState>(m + j),
           vv = ld4_state<kStreamState>(v + j), vh = ld4_state<kStreamState>(vhat + j);
    for (int q = tid; q < kBatch * kWave; q += kThreads) (&kept[0][0])[q] = 0u;
    if (r == 0) {
        // lane i: where worker i keeps the quarter's candidates, and its threshold
        uint32_t count = 0;
        if (lane < ge.n) {
            const uint4 rec = tile_dir[(int64_t)lane * ge.n_tiles + t];
            const TkWorker *wk = ws + lane;
            const uint32_t c[4] = {rec.y & 0xffffu, rec.y >> 16, rec.z & 0xffffu, rec.z >> 16};
            uint32_t at = rec.x;
            for (int q = 0; q < w; ++q) at += c[q];
            count = c[w];
            start[lane] = at;
            tc[lane] = wk->tc;
            const SelKey sk = sel_key_of(ge.rand, wk->step_word, lane);
            key_a[lane] = sk.a;
            key_b[lane] = sk.b;
        }
        const uint32_t incl = wave_scan(count);
        if (lane < ge.n) upto[lane + 1] = incl;
        if (lane == 0) upto[0] = 0u;
    }
    __syncthreads();
    const uint32_t total = upto[ge.n];
    // The worker of entry q < total of the quarter is the last one whose entries start at or before it (upto[ge.n] = total lies
    // beyond every q).  A thread's first entries are looked for together, those of a batch among its workers.
    auto last_before = [&](int i, int bit, uint32_t q) { return upto[min(i + bit, ge.n)] <= q ? i + bit : i; };
    auto owner = [&](uint32_t q, int w0) {
        int i = w0;
#pragma unroll
        for (int bit = 4; bit > 0; bit >>= 1) i = last_before(i, bit, q);
        return i;
    };
    static_assert(kBatch <= 8, "three steps");
    auto fetch = [&](uint32_t q, int i) { return cand[worker_base(ge, i) + start[i] + (q - upto[i])]; };
    auto is_kept = [&](const uint2 &e, int i) {
        const SelKey sk = {ge.rand.on, key_a[i], key_b[i]};
        return composite(sel_key(sk, __uint_as_float(e.y), e.x), e.x, ge.idx_bits) >= tc[i];
    };
    auto put = [&](const uint2 &e, int u) {
        const uint32_t l = e.x - base;
        val[u][(l >> 10) * 256u + (l & 255u)] = __uint_as_float(e.y);
        atomicOr(&kept[u][(l >> 2) & 63u], 1u << ((l >> 10) * 4u + (l & 3u)));
    };
    uint2 e[kShortHeld];
    int of[kShortHeld];
#pragma unroll
    for (int s = 0; s < kShortHeld; ++s) of[s] = 0;
    for (int bit = ge.n > 1 ? 1 << (31 - __clz(ge.n - 1)) : 0; bit > 0; bit >>= 1)      // from the greatest power of two below n
#pragma unroll
        for (int s = 0; s < kShortHeld; ++s) of[s] = last_before(of[s], bit, tid + s * kThreads);
#pragma unroll
    for (int s = 0; s < kShortHeld; ++s) {
        const uint32_t q = tid + s * kThreads;
        if (q >= total) of[s] = -1;
        e[s] = make_uint2(0u, 0u);
        if (of[s] >= 0) e[s] = fetch(q, of[s]);
    }
#pragma unroll
    for (int s = 0; s < kShortHeld; ++s)
        if (of[s] >= 0 && !is_kept(e[s], of[s])) of[s] = -1;
    // entries beyond those: the first of each thread in the batch that begins with worker w0 is read a batch ahead
    uint32_t more = 0;
    int more_of = -1;
    uint2 more_e = make_uint2(0u, 0u);
    auto read_ahead = [&](int w0) {
        more = max(upto[w0], (uint32_t)(kShortHeld * kThreads)) + tid;
        more_of = more < upto[min(w0 + kBatch, ge.n)] ? owner(more, w0) : -1;
        if (more_of >= 0) more_e = fetch(more, more_of);
    };
    read_ahead(0);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int w0 = 0; w0 < ge.n; w0 += kBatch) {
        const int nw = min(kBatch, ge.n - w0);
        if (w0) {
            __syncthreads();                                 // the bits of the batch before have been read
            for (int q = tid; q < kBatch * kWave; q += kThreads) (&kept[0][0])[q] = 0u;
            __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < kShortHeld; ++s)
            if ((uint32_t)(of[s] - w0) < (uint32_t)nw) put(e[s], of[s] - w0);
        if (more_of >= 0 && is_kept(more_e, more_of)) put(more_e, more_of - w0);
        for (uint32_t q = more + kThreads; q < upto[w0 + nw]; q += kThreads) {
            const int i = owner(q, w0);
            const uint2 x = fetch(q, i);
            if (is_kept(x, i)) put(x, i - w0);
        }
        if (w0 + kBatch < ge.n) read_ahead(w0 + kBatch);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (u < nw) {
                const uint32_t bits = kept[u][lane] >> (4 * r);
                const float4 x = ld4(&val[u][256 * r + 4 * lane]);      // anything where nothing was kept
                if (bits & 1u) acc[0] = fadd(acc[0], x.x);
                if (bits & 2u) acc[1] = fadd(acc[1], x.y);
                if (bits & 4u) acc[2] = fadd(acc[2], x.z);
                if (bits & 8u) acc[3] = fadd(acc[3], x.w);
            }
        }
    }
    const float4 gbar = make_float4(fdiv(acc[0], p.n_workers), fdiv(acc[1], p.n_workers), fdiv(acc[2], p.n_workers),
                                    fdiv(acc[3], p.n_workers));
    const float4 vh0 = vh;
    amsgrad_update4(th, mm, vv, vh, gbar, p);
    st4_state<kStreamState>(theta + j, th);
    st4_state<kStreamState>(m + j, mm);
    st4_state<kStreamState>(v + j, vv);
    // with a sparse average vhat = max(vhat, v) moves at few coordinates (v only decays elsewhere)
    st4_if_changed<kStreamState>(vhat + j, vh, vh0);
}

// ---------------------------------------------------------------------------------------------
// How the workgroups of tk_hist and tk_compact share a worker's candidates: bx (blockIdx.x) = slice *
// parts + part, and a part is a contiguous piece of the slice's region.
struct Piece {
    int slice;
    uint32_t q0, q1;     // entries [q0, q1) of the region
};
__device__ __forceinline__ Piece piece_of(const TkGeom &ge, const uint32_t *__restrict__ cursor, int worker, int bx)
{
    Piece p;
    p.slice = bx / ge.parts;
    const uint32_t part = bx % ge.parts;
    const uint32_t count = min(cursor[(worker * ge.slices + p.slice) * kCursorStride], ge.region_cap);
    const uint32_t chunk = (count + ge.parts - 1) / ge.parts;
    p.q0 = min(part * chunk, count);
    p.q1 = min(p.q0 + chunk, count);
    return p;
}

// ---------------------------------------------------------------------------------------------
// How a kernel forms the vector that is compressed again from what is stored:
//   kSrcStored  the stored x itself (error feedback)
//   kSrcGrad    g - ghat_i, a = g (rows of d floats, any 4-byte alignment), b = ghat_i (CD-Adam workers)
//   kSrcDiff    a - b, both padded rows (CD-Adam server: ghat - gtilde)
//   kSrcGradOnly  a = g itself (naive compression)
enum { kSrcStored = 0, kSrcGrad = 1, kSrcDiff = 2, kSrcGradOnly = 3 };

// The coordinates j .. j + 3 of vector i (j a multiple of 4) as they are stored, and their values.  a: for kSrcGrad /
// kSrcGradOnly the gradients (elements of type G), else padded float rows; brow: row i of b.
template <int kSrc, typename G>
struct Source4 {
    static constexpr bool kGrad = kSrc == kSrcGrad || kSrc == kSrcGradOnly, kTwo = kSrc == kSrcGrad || kSrc == kSrcDiff;
    GradRaw<std::conditional_t<kGrad, G, float>> a;
    float4 b;
    __device__ __forceinline__ void load(const void *__restrict__ av, int i, const TkGeom &ge, const float *__restrict__ brow,
                                         uint32_t j, uint32_t d)
    {
        if constexpr (kGrad) {
            a = load_raw4<false>(static_cast<const G *>(av) + (int64_t)i * ge.d, j, d);
        } else {
            const float4 x = ld4(static_cast<const float *>(av) + (int64_t)i * ge.ld + j);
            a.v = {x.x, x.y, x.z, x.w};
        }
        if (kTwo) b = ld4(brow + j);
    }
    __device__ __forceinline__ float4 value() const
    {
        const float4 x = widen4(a);
        return kTwo ? make_float4(fsub(x.x, b.x), fsub(x.y, b.y), fsub(x.z, b.z), fsub(x.w, b.w)) : x;
    }
};

// The 16 values of this thread in the tile at `base` (coordinates base + 4 (tid + 256 r) + c).
template <int kSrc, typename G>
__device__ __forceinline__ void load_source_tile(float (&x)[4][4], const void *__restrict__ a, int i, const TkGeom &ge,
                                                 const float *__restrict__ brow, uint32_t base, uint32_t d)
{
    Source4<kSrc, G> s[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) s[r].load(a, i, ge, brow, base + 4 * (threadIdx.x + kThreads * r), d);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float4 v = s[r].value();
        x[r][0] = v.x;
        x[r][1] = v.y;
        x[r][2] = v.z;
        x[r][3] = v.w;
    }
}

// Which way a worker's selection goes in this step, from what the listing pass left (the same test in tk_hist and
// tk_compact, which see the same cursors and flags):
//   kCaseListed    every element at or above the guess is listed and there are at least k of them: the k-th largest
//                  is a candidate, the candidate histograms locate it;
//   kCaseZeroTail  error feedback with magnitude keys, a guess of 0 (every non-zero element is listed) and fewer
//                  than k candidates: the k-th largest is a zero (see zero_tail_threshold);
//   kCaseMiss      the guess was too high (always on the first step, else when the threshold fell through the slack),
//                  or a candidate region was full: nothing below the guess is known, the whole vector is counted.
enum { kCaseListed = 0, kCaseZeroTail = 1, kCaseMiss = 2 };
template <int kSrc>
__device__ __forceinline__ int selection_case(const TkGeom &ge, uint32_t total, uint32_t guess, bool overflow)
{
    if (total >= ge.k && !overflow) return kCaseListed;
    if (kSrc == kSrcStored && !ge.rand.on && guess == 0u && !overflow) return kCaseZeroTail;
    return kCaseMiss;
}

// Number of candidates of worker i = sum of its region cursors; every wavefront adds them up for itself.
__device__ __forceinline__ uint32_t candidates_listed(const TkGeom &ge, const uint32_t *__restrict__ cursor, int i)
{
    uint32_t c = 0;
    for (int q = threadIdx.x & 63; q < ge.slices; q += kWave) c += cursor[(i * ge.slices + q) * kCursorStride];
    return scan_total(wave_scan(c));
}

// First coarse bin of the window whose fine bins are counted: the guess's, but no more than kWindowBelow fine bins below the
// previous threshold.  With a wide slack (after a fall, or for Rand-k) a window that began at the guess ended before the
// thresholds of the next steps, and the threshold bin held 64 times the elements: CD-Adam n = 8, d = 11.2 M bf16, on two
// batches in turn, tk_resolve took 36 us in every second step and takes 6.  224 = half of the window less half a coarse bin:
// with its start rounded down to a coarse bin, the window reaches 224 to 287 fine bins to either side of the previous threshold.
// Candidates below the window are counted in a few coarse bins, which it is there to avoid; what that costs where the slack is
// wide is less than what their fine bins cost (tk_hist, us, window from the guess on / this: CD-Adam as above 9.5 / 8.6, Rand-k n = 16,
// d = 1.2 M with 25 % kept 19.8 / 18.3, n = 8, d = 5 M with 20 % kept 36.4 / 31.4, 1 % kept f16 3.9 / 4.0; the candidates' loads
// changed in between as well).
// So coarse bins may lie between the guess and the window, and the guess's own is listed only from the guess on: a coarse
// prefix does not mean that all elements of the bin are among the candidates, and the bin's lower edge, which lies below the
// guess, is no threshold (tk_compact's `whole`).  The digits below such a prefix (kFirstBits bits and more) are narrower than
// a fine bin, and no candidate lies below the guess: the lower edge of the digit of the k-th largest does not either.
constexpr uint32_t kWindowBelow = 224;
__device__ __forceinline__ uint32_t window_start(uint32_t guess, uint32_t last)
{
    if (last != kNoGuess && last > guess + kWindowBelow) guess = last - kWindowBelow;
    return guess >> (kShift1 - kFineShift);
}

// First kernel of the selection.  Grid (slices * parts, n).
// Usual case (kCaseListed): histograms of the candidates of a worker - the fine bins of the kWindowCoarse coarse bins
// from window_start on, and the coarse bins of the candidates outside that window (those inside it would
// draw most LDS atomics to eight words; tk_compact adds them up from the fine bins).  Loads are issued four at a
// time, without a branch around them (past the end the last element is read again): in one the compiler waits for each load
// before it issues the next.
// After a miss (kCaseMiss) the workgroups of the worker count the whole vector, re-formed from what is stored
// (a, b: see load_source_tile), into the worker's full coarse histogram instead; tk_compact takes the coarse bin of
// the k-th largest from it and lists again.  Bin 0 (zeros and the smallest denormals) is not counted there but
// taken as the remainder: in a sparse vector it would draw most LDS atomics of a tile to one word.
template <int kSrc, typename G>
__global__ __launch_bounds__(kThreads) void tk_hist(TkGeom ge, const TkWorker *__restrict__ ws,
                                                    const uint2 *__restrict__ cand,
                                                    const uint32_t *__restrict__ cursor,
                                                    uint32_t *__restrict__ hist1, uint32_t *__restrict__ histf,
                                                    uint32_t *__restrict__ hist_full, const void *__restrict__ a,
                                                    const float *__restrict__ b)
{
    __shared__ uint32_t lh[kBins1];
    __shared__ uint32_t lf[kFineWindow];
    const int i = blockIdx.y;
    const int tid = threadIdx.x;
    const uint32_t guess = ws[i].guess, last = ws[i].last_fine;
    const uint32_t total = candidates_listed(ge, cursor, i);
    const int which = selection_case<kSrc>(ge, total, guess, ws[i].overflow != 0u);
    if (which == kCaseZeroTail) return;
    const Piece pc = piece_of(ge, cursor, i, (int)blockIdx.x);
    if (which == kCaseListed && pc.q0 >= pc.q1) return;
    const SelKey sk = sel_key_of(ge.rand, ge.rand.step_now, i);
    for (int q = tid; q < kBins1; q += kThreads) lh[q] = 0;
    if (which == kCaseMiss) {
        __syncthreads();
        const uint32_t d = (uint32_t)ge.d;
        const float *brow = (kSrc == kSrcGrad || kSrc == kSrcDiff) ? b + (int64_t)i * ge.ld : nullptr;
        for (int t = blockIdx.x; t < ge.n_tiles; t += gridDim.x) {
            const uint32_t base = (uint32_t)t * kTile;
            float x[4][4];
            load_source_tile<kSrc, G>(x, a, i, ge, brow, base, d);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t j = base + 4 * (tid + kThreads * r) + c;
                    const uint32_t bin = sel_key(sk, x[r][c], j) >> kShift1;
                    if (bin != 0 && j < d) atomicAdd(&lh[bin], 1u);
                }
        }
        __syncthreads();
        for (int q = tid; q < kBins1; q += kThreads) {
            const uint32_t c = lh[q];
            if (c) atomicAdd(hist_full + (int64_t)i * kBins1 + q, c);
        }
        return;
    }
    for (int q = tid; q < kFineWindow; q += kThreads) lf[q] = 0;
    __syncthreads();
    const uint32_t wbase = window_start(guess, last) * kFinePerCoarse;
    const uint2 *src = cand + region_base(ge, i, pc.slice);
    for (uint32_t qb = pc.q0; qb < pc.q1; qb += 4 * kThreads) {
        uint2 y[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t q = qb + u * kThreads + tid;
            y[u] = src[min(q, pc.q1 - 1u)];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (qb + u * kThreads + tid < pc.q1) {
                const uint32_t fine = sel_key(sk, __uint_as_float(y[u].y), y[u].x) >> kFineShift;
                if (fine - wbase < (uint32_t)kFineWindow)
                    atomicAdd(&lf[fine - wbase], 1u);
                else
                    atomicAdd(&lh[fine >> (kShift1 - kFineShift)], 1u);
            }
        }
    }
    __syncthreads();
    for (int b1 = tid; b1 < kBins1; b1 += kThreads) {
        const uint32_t c = lh[b1];
        if (c) atomicAdd(hist1 + (int64_t)i * kBins1 + b1, c);
    }
    for (int q = tid; q < kFineWindow; q += kThreads)
        if (lf[q]) atomicAdd(histf + (int64_t)i * kFineWindow + q, lf[q]);
}

// Second kernel of the selection: the leading digits of Tc, and the elements they leave.  Grid (at least
// slices * parts, n).
// Usual case (kCaseListed): every workgroup finds the coarse and (if the window covers it) fine bin of the k-th
// largest from the candidate histograms for itself - 10 KB from the caches and one scan, about a microsecond, where a
// launch of its own took six - and copies the candidates of its piece that carry this prefix, as comp values, to the
// dense storage.  Each wavefront takes a quarter of the workgroup's piece and writes its hits from the start of that
// quarter onwards (as many slots as it reads, so it cannot overflow), and records {start, count} relative to the
// worker's first region; no atomics, tk_resolve walks the records.  While copying, the workgroup counts the next
// kFirstBits bits of comp below the prefix (hist2: [n][kBinsFirst], added to with atomics, emptied by tk_resolve) and
// every wavefront notes which of those digits occur in its piece (piece_bits: kPieceWords words per piece, written
// whole).  Nothing is copied where the threshold needs no further digit.  The histograms are cleared by tk_resolve.
// After a miss tk_hist has counted the whole vector into the worker's full coarse histogram: every workgroup takes
// the coarse bin of the k-th largest from it and lists the elements in that bin or above, tile by tile, into the
// worker's regions - through the second set of cursors (cursor_b, all zero here), since the first still holds the
// counts this kernel's workgroups decide by - and count the first digit in that bin as above.  The worker is flagged
// `relisted`: tk_resolve then takes the elements from these lists (no dense pieces exist) and clears both sets.  A region that fills up there as well sets
// overflow2: tk_resolve then selects without lists (exact_select).
template <int kSrc, typename G>
__global__ __launch_bounds__(kThreads) void tk_compact(TkGeom ge, TkWorker *__restrict__ ws,
                                                       const uint32_t *__restrict__ hist1,
                                                       const uint32_t *__restrict__ histf,
                                                       const uint32_t *__restrict__ cursor,
                                                       uint32_t *__restrict__ cursor_b,
                                                       const uint32_t *__restrict__ hist_full,
                                                       const void *__restrict__ a, const float *__restrict__ b,
                                                       uint2 *__restrict__ cand, uint4 *__restrict__ tile_dir,
                                                       uint64_t *__restrict__ dense, uint2 *__restrict__ dense_dir,
                                                       uint32_t *__restrict__ hist2, uint32_t *__restrict__ piece_bits)
{
    __shared__ uint32_t lf[kFineWindow];
    __shared__ uint32_t win[kWindowCoarse];
    __shared__ uint32_t lh2[kBinsFirst];
    __shared__ uint32_t bits[kThreads / kWave][kPieceWords];
    __shared__ uint32_t part[kThreads / kWave];
    __shared__ uint32_t res[3];
    __shared__ uint32_t sh[9];
    static_assert(kBins1 == 8 * kThreads && kFineWindow == 2 * kThreads, "bins owned per thread");
    static_assert(kFinePerCoarse == kWave && kWindowCoarse == 2 * (kThreads / kWave), "fine bins of two coarse bins per wavefront");
    const int i = blockIdx.y;
    const int bx = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int per = ge.slices * ge.parts;
    // What the usual case needs goes out before anything waits: this thread's coarse bins, two fine bins (of the
    // window's coarse bins `wave` and `wave + 4`), and the size of the workgroup's piece
    const uint4 own0 = *reinterpret_cast<const uint4 *>(hist1 + (int64_t)i * kBins1 + 8 * tid);
    const uint4 own1 = *reinterpret_cast<const uint4 *>(hist1 + (int64_t)i * kBins1 + 8 * tid + 4);
    const uint32_t f0 = histf[(int64_t)i * kFineWindow + tid], f1 = histf[(int64_t)i * kFineWindow + kThreads + tid];
    const Piece pc = piece_of(ge, cursor, i, min(bx, per - 1));
    const uint32_t guess = ws[i].guess, last = ws[i].last_fine;
    const bool overflow = ws[i].overflow != 0u;
    {
        lf[tid] = f0;
        lf[kThreads + tid] = f1;
        const uint32_t s0 = scan_total(wave_scan(f0)), s1 = scan_total(wave_scan(f1));
        if (lane == 0) {
            win[wave] = s0;
            win[wave + kThreads / kWave] = s1;
        }
        for (int q = tid; q < kBinsFirst; q += kThreads) lh2[q] = 0;
        if (lane < kPieceWords) bits[wave][lane] = 0;
    }
    const uint32_t total = candidates_listed(ge, cursor, i);
    __syncthreads();                                                         // what was put into LDS
    const int which = selection_case<kSrc>(ge, total, guess, overflow);
    const SelKey sk = sel_key_of(ge.rand, ge.rand.step_now, i);

    if (which == kCaseListed) {
        if (bx >= per) return;                      // workgroups beyond the pieces are there for the lists after a miss
        const uint32_t wb = window_start(guess, last);            // first coarse bin of the fine window
        uint32_t own[8] = {own0.x, own0.y, own0.z, own0.w, own1.x, own1.y, own1.z, own1.w};
#pragma unroll
        for (int q = 0; q < 8; ++q) {               // the window's coarse bins are counted in the fine histogram alone
            const uint32_t at = 8 * tid + q - wb;
            if (at < (uint32_t)kWindowCoarse) own[q] += win[at];
        }
        find_rank_owned(own, part, res, ge.k);
        uint32_t prefix = res[0];                   // coarse bin of the k-th largest
        uint32_t pshift = kShift1;
        uint32_t rank = ge.k - res[1];
        uint32_t count = res[2];
        if (prefix - wb < (uint32_t)kWindowCoarse) {
            // the fine histogram covers this coarse bin: pick the fine bin as well (every wavefront for itself)
            const uint32_t c = lf[(prefix - wb) * kFinePerCoarse + lane];
            const uint32_t incl = wave_scan(c);
            const uint32_t suffix = scan_total(incl) - incl + c;      // candidates of this coarse bin in fine bins >= lane
            const uint64_t reach = __ballot(suffix >= rank);      // lane 0 reaches: suffix(0) = count >= rank
            const int top = reach ? 63 - __builtin_clzll(reach) : 0;
            count = (uint32_t)__shfl((int)c, top, kWave);
            rank -= (uint32_t)__shfl((int)suffix, top, kWave) - count;
            prefix = (prefix << (kShift1 - kFineShift)) | (uint32_t)top;
            pshift = kFineShift;
        }
        // every element with this prefix is kept: only where all of them were listed (see window_start)
        const bool whole = count == rank && (pshift == (uint32_t)kFineShift || prefix * kFinePerCoarse >= guess);
        if (bx == 0 && tid == 0) {
            ws[i].prefix = prefix;
            ws[i].pshift = pshift;
            ws[i].rank = rank;
            ws[i].whole = whole ? 1u : 0u;
            ws[i].relisted = 0u;
        }
        if (whole) return;
        const FirstDigit fd = first_digit(ge, pshift);
        const uint32_t quarter = (pc.q1 - pc.q0 + 3) / 4;
        const uint32_t w0 = min(pc.q0 + wave * quarter, pc.q1), w1 = min(w0 + quarter, pc.q1);
        const int64_t rbase = region_base(ge, i, pc.slice);
        const uint2 *src = cand + rbase;
        uint64_t *out = dense + rbase + w0;
        uint32_t kept = 0;
        for (uint32_t qb = w0; qb < w1; qb += 4 * kWave) {
            uint2 c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t q = qb + u * kWave + lane;
                c[u] = src[min(q, w1 - 1u)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t key = sel_key(sk, __uint_as_float(c[u].y), c[u].x);
                const bool hit = qb + u * kWave + lane < w1 && (key >> pshift) == prefix;
                const uint32_t slot = wave_append(hit, kept);
                if (hit) {
                    const uint64_t comp = composite(key, c[u].x, ge.idx_bits);
                    out[slot] = comp;
                    const uint32_t digit = digit_of(fd, comp);
                    atomicAdd(&lh2[digit], 1u);
                    atomicOr(&bits[wave][digit >> 5], 1u << (digit & 31u));
                }
            }
        }
        const int64_t rec = ((int64_t)i * per + bx) * 4 + wave;
        if (lane == 0) dense_dir[rec] = make_uint2((uint32_t)(rbase - worker_base(ge, i)) + w0, kept);
        // the piece's bitmap, written whole every step (the wavefront reads back its own LDS atomics)
        if (lane < kPieceWords) piece_bits[rec * kPieceWords + lane] = bits[wave][lane];
        __syncthreads();
        for (int q = tid; q < kBinsFirst; q += kThreads) {
            const uint32_t c = lh2[q];
            if (c) atomicAdd(hist2 + (int64_t)i * kBinsFirst + q, c);
        }
        return;
    }

    if (which == kCaseZeroTail) {
        // all candidates are kept; tk_resolve places the threshold among the zeros, which are ordered by index
        // alone, from the zero counts of the tiles
        if (bx != 0) return;
        if (tid == 0) {
            ws[i].prefix = 0u;
            ws[i].pshift = kShift1;
            ws[i].rank = ge.k - total;          // so many zeros are kept, the lowest indices first
            ws[i].whole = kZeroTail;
            ws[i].relisted = 0u;
        }
        return;
    }

    // after a miss: the coarse bin of the k-th largest from the full histogram, and the lists anew
    const uint32_t d = (uint32_t)ge.d;
    {
        uint32_t own[8];
        uint32_t counted = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            own[q] = hist_full[(int64_t)i * kBins1 + 8 * tid + q];
            counted += own[q];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) counted += __shfl_xor(counted, off, kWave);
        if (lane == 0) sh[wave] = counted;
        __syncthreads();
        if (tid == 0) own[0] = d - (sh[0] + sh[1] + sh[2] + sh[3]);   // bin 0 is the remainder
        find_rank_owned(own, part, res, ge.k);             // the histogram holds all d >= k elements
    }
    const uint32_t prefix = res[0];
    if (bx == 0 && tid == 0) {
        ws[i].prefix = prefix;
        ws[i].pshift = kShift1;
        ws[i].rank = ge.k - res[1];
        ws[i].whole = (res[2] == ge.k - res[1]) ? 1u : 0u;
        ws[i].relisted = 1u;
    }
    const float *brow = (kSrc == kSrcGrad || kSrc == kSrcDiff) ? b + (int64_t)i * ge.ld : nullptr;
    for (int t = bx; t < ge.n_tiles; t += gridDim.x) {
        const uint32_t base = (uint32_t)t * kTile;
        float x[4][4];
        load_source_tile<kSrc, G>(x, a, i, ge, brow, base, d);
        // count first, then write straight from the registers into the space taken: no staging lists
        uint32_t count = 0, zeros = 0, hits = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t j = base + 4 * (tid + kThreads * r) + c;
                const uint32_t key = sel_key(sk, x[r][c], j);
                bool hit = j < d && (key >> kShift1) >= prefix;
                if (kSrc == kSrcStored && !sk.on) {          // zeros are counted, not listed (as in tk_pass1)
                    const bool zero = j < d && mag_key(x[r][c]) == 0u;
                    zeros += (uint32_t)__popcll(__ballot(zero));
                    hit = hit && !zero;
                }
                // the digit below the prefix, as in the usual case
                if (hit && (key >> kShift1) == prefix)
                    atomicAdd(&lh2[(key >> (kShift1 - kFirstBits)) & (uint32_t)(kBinsFirst - 1)], 1u);
                count += (uint32_t)__popcll(__ballot(hit));
                hits |= (hit ? 1u : 0u) << (r * 4 + c);
            }
        take_tile_space(count, zeros, sh, ge, i, t, cursor_b, tile_dir, &ws[i].overflow2);
        uint32_t at = sh[4];
        if (at != kNoSpace) {
            for (int w = 0; w < wave; ++w) at += sh[w];
            uint2 *dst = cand + worker_base(ge, i);
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool hit = (hits >> (r * 4 + c)) & 1u;
                    const uint32_t slot = wave_append(hit, at);
                    if (hit) dst[slot] = make_uint2(base + 4 * (tid + kThreads * r) + c, __float_as_uint(x[r][c]));
                }
        }
        __syncthreads();   // sh is reused by the next tile
    }
    __syncthreads();
    for (int q = tid; q < kBinsFirst; q += kThreads) {
        const uint32_t c = lh2[q];
        if (c) atomicAdd(hist2 + (int64_t)i * kBinsFirst + q, c);
    }
}

// ---------------------------------------------------------------------------------------------
// One workgroup of 1024 threads per worker: the digits of Tc below the prefix, over the pieces
// tk_compact filled (slices * parts * 4 <= 2 * kResolveThreads of them).  Hands the next step its
// guess and empties the worker's region cursors for it.
constexpr int kMaxPieces = 2048;   // slices * parts * 4 never exceeds this (the host picks parts accordingly)
constexpr int kFew = 256;         // at most this many elements are ranked directly instead of by further digits
                                  // (1024 measured slower: ranking a thousand elements against each other costs
                                  // more than one more digit over a threshold bin of a few thousand)
static_assert(kMaxPieces <= 2 * kResolveThreads, "two pieces per thread in the prefix sum");

constexpr int kScanUnroll = 4;    // independent loads per thread in the scans of the dense set
constexpr int kStaged = 8192;     // elements under the first digit of Tc that are collected in LDS for the further digits

// LDS of the digit search, in tk_resolve and tk_small_select.
struct ResolveLds {
    uint32_t lh[kBins2];
    uint32_t part[kResolveThreads / kWave];
    uint32_t res[4];
    uint64_t few[kFew];
    uint32_t n_few;
    uint64_t tc_sh;
};

// The comp value of 1-based rank `rank` from the top among the n <= kFew in L.few (unique; a barrier after they were put there);
// ends with a barrier.
__device__ __forceinline__ uint64_t rank_few(uint32_t n, uint32_t rank, ResolveLds &L)
{
    if (threadIdx.x < n) {
        const uint64_t mine = L.few[threadIdx.x];
        uint32_t greater = 0;
        for (uint32_t u = 0; u < n; ++u) greater += L.few[u] > mine ? 1u : 0u;
        if (greater + 1 == rank) L.tc_sh = mine;              // comp values are unique: exactly one thread
    }
    __syncthreads();
    return L.tc_sh;
}

// The digits of Tc below `prefix` (which leaves s_hi low bits of comp open), 12 bits at a time, over the
// cnt comp values that fetch(q, comp) delivers kScanUnroll at a time (comp[u] = element q[u], anything for
// q[u] >= cnt; q ascends with u), of which the one of 1-based rank `rank` (from the top) among those that
// carry the prefix is wanted.  Once at most kFew elements carry the prefix they are fetched and
// ranked against each other directly.  All threads of the workgroup call this; returns Tc.
// kWholeBins: a digit whose bin holds exactly the elements still wanted ends the search with the bin's lower edge as
// Tc - right when every element of the vector that could fall into that bin is among the cnt delivered (a digit of
// tk_compact's threshold bin lies in one fine bin, and those are listed whole), wrong when the elements are only those above some bound that may cut the bin
// (the list of tk_small_select): then the search goes on to the k-th largest comp value itself.
template <bool kWholeBins = true, class Fetch>
__device__ __forceinline__ uint64_t resolve_digits(Fetch fetch, uint32_t cnt, uint64_t prefix, uint32_t rank, int s_hi,
                                                   ResolveLds &L)
{
    const int tid = threadIdx.x;
    const int nt = (int)blockDim.x;
    uint64_t tc = prefix << s_hi;
    bool done = false;
    while (!done) {
        const int s_lo = max(s_hi - kDigitBits, 0);
        const uint32_t mask = (1u << (s_hi - s_lo)) - 1u;
        for (int b = tid; b < kBins2; b += nt) L.lh[b] = 0;
        __syncthreads();
        for (uint32_t qb = 0; qb < cnt; qb += kScanUnroll * nt) {
            uint32_t q[kScanUnroll];
            uint64_t comp[kScanUnroll];
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) q[u] = qb + u * nt + tid;
            fetch(q, comp);                                     // independent loads: all in flight at once
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u)
                if (q[u] < cnt && (comp[u] >> s_hi) == prefix)
                    atomicAdd(&L.lh[(uint32_t)(comp[u] >> s_lo) & mask], 1u);
        }
        __syncthreads();
        find_rank_bin<kBins2>(L.lh, L.part, L.res, rank);
        if (!L.res[3]) break;                                  // cannot happen: rank <= matching elements
        prefix = (prefix << (s_hi - s_lo)) | L.res[0];
        rank -= L.res[1];
        const uint32_t left = L.res[2];                        // elements that carry the new prefix
        s_hi = s_lo;
        if (s_lo == 0 || (kWholeBins && left == rank)) {       // last digit, or all under this prefix are kept
            done = true;
            tc = prefix << s_lo;
        } else if (left <= (uint32_t)min(kFew, nt)) {
            if (tid == 0) L.n_few = 0;
            __syncthreads();
            for (uint32_t qb = 0; qb < cnt; qb += kScanUnroll * nt) {
                uint32_t q[kScanUnroll];
                uint64_t comp[kScanUnroll];
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u) q[u] = qb + u * nt + tid;
                fetch(q, comp);
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u)
                    if (q[u] < cnt && (comp[u] >> s_hi) == prefix)
                        L.few[atomicAdd(&L.n_few, 1u)] = comp[u];
            }
            __syncthreads();
            done = true;
            tc = rank_few(left, rank, L);
        }
        __syncthreads();
    }
    return tc;
}

// Records the finished selection of a worker and prepares the next step's guess: a few fine bins
// below this threshold - at least twice the distance the threshold just fell (a rising threshold needs
// no slack), never less than kMinSlack, shrinking by one bin per quiet step, doubled after a miss.
// w: the record as the step found it (its slack and last threshold bin).  The flags of the running step are
// cleared for the next one.  One thread calls this.
__device__ __forceinline__ void finish_worker(TkWorker *ws, int i, const TkWorker &w, uint64_t tc, const TkGeom &ge,
                                              bool missed)
{
    ws[i].tc = tc;
    ws[i].step_word = ge.rand.step_now;
    const uint32_t fine = (uint32_t)(tc >> ge.idx_bits) >> kFineShift;
    const uint32_t fell = (w.last_fine != kNoGuess && w.last_fine > fine) ? w.last_fine - fine : 0u;
    uint32_t slack = missed ? w.slack * 2u : w.slack - 1u;
    slack = max(slack, 2u * fell + 2u);
    slack = min(max(slack, max(kMinSlack, ge.rand.min_slack)), kMaxSlack);
    ws[i].slack = slack;
    ws[i].last_fine = fine;
    ws[i].guess = fine > slack ? fine - slack : 0u;
    ws[i].overflow = 0u;
    ws[i].overflow2 = 0u;
}

// Exclusive prefix sum of one value per thread over the 1024 threads of tk_resolve; returns the exclusive sum,
// leaves the total in *total_sh.  part: 16 LDS words.  Two barriers.
__device__ __forceinline__ uint32_t resolve_scan(uint32_t v, uint32_t *part, uint32_t *total_sh)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t incl = wave_scan(v);
    __syncthreads();                       // readers of an earlier part are done
    if (lane == kWave - 1) part[wave] = incl;
    __syncthreads();
    const uint32_t before = waves_before(part, wave);
    if (threadIdx.x == kResolveThreads - 1) *total_sh = before + incl;
    return before + incl - v;
}

// Error feedback with fewer than k non-zero coordinates: the threshold is the comp value of the R-th zero of
// the stored row in index order (zeros tie, the lower index wins), found from the tiles' zero counts: first
// the tile that holds it, then its place inside that tile.  All kResolveThreads threads call this; R >= 1 and
// the row holds at least R zeros below d.
__device__ __forceinline__ uint64_t zero_tail_threshold(const uint4 *__restrict__ dir_row, const float *__restrict__ xrow,
                                                        const TkGeom &ge, uint32_t R, ResolveLds &L)
{
    const int tid = threadIdx.x;
    if (tid == 0) {                              // what is read below if the counts held fewer than R zeros
        L.res[0] = 0u;
        L.res[1] = 0u;
        L.tc_sh = (1ull << ge.idx_bits) - 1ull;
    }
    const int chunk = (ge.n_tiles + kResolveThreads - 1) / kResolveThreads;
    const int t0 = min(tid * chunk, ge.n_tiles), t1 = min(t0 + chunk, ge.n_tiles);
    uint32_t mine = 0;
    for (int t = t0; t < t1; ++t) mine += dir_row[t].w;
    uint32_t before = resolve_scan(mine, L.part, &L.res[3]);
    if (before < R && R <= before + mine) {
        for (int t = t0; t < t1; ++t) {
            const uint32_t z = dir_row[t].w;
            if (before + z >= R) {
                L.res[0] = (uint32_t)t;           // the tile of the R-th zero ...
                L.res[1] = R - before;            // ... which is this tile's res[1]-th zero
                break;
            }
            before += z;
        }
    }
    __syncthreads();
    const uint32_t base = L.res[0] * (uint32_t)kTile, r = L.res[1];
    // the tile in coordinate order: thread tid holds the coordinates base + 4 tid .. + 3 (padding is not counted)
    const float4 v = ld4(xrow + base + 4 * tid);
    const float x[4] = {v.x, v.y, v.z, v.w};
    uint32_t zc = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) zc += (base + 4 * tid + c < (uint32_t)ge.d && mag_key(x[c]) == 0u) ? 1u : 0u;
    uint32_t seen = resolve_scan(zc, L.part, &L.res[3]);
    if (seen < r && r <= seen + zc) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (base + 4 * tid + c < (uint32_t)ge.d && mag_key(x[c]) == 0u && ++seen == r)
                L.tc_sh = ((1ull << ge.idx_bits) - 1ull) - (uint64_t)(base + 4 * tid + c);   // key part 0
        }
    }
    __syncthreads();
    return L.tc_sh;
}

// ---------------------------------------------------------------------------------------------
// Selection without lists, for a vector whose candidates fit no region even when listed anew (so many elements
// share the leading bits of the k-th largest that only the whole composite key tells them apart - all-equal
// input is the extreme).  The worker's workgroup of tk_resolve does it alone: the digits of Tc by counting over
// the whole vector, re-formed element by element from what is stored (kDigitBits bits per sweep), then one more
// sweep that lists exactly the kept elements - k of them, which always fit: a worker's regions hold at least 8 k
// entries in all, and this list is written as one run from the worker's first region (no cursors; a tile's
// record holds its offset in that run, its candidates stand by owning wavefront as everywhere).  Slow - one
// compute unit reads the vector up to six times - and meant to be: it only has to be right.
//
// How the vector is re-formed (src: kSrcStored ... kSrcGradOnly; gtype: element type of the gradients, 0 fp32,
// 1 bfloat16, 2 half) is decided at run time here: one scalar load per element and operand.
struct ExactSource {
    int32_t src, gtype;
    const void *a;
    const float *b;
};
__device__ __forceinline__ float exact_value(const ExactSource &e, const TkGeom &ge, int i, uint32_t j)
{
    float av;
    if (e.src == kSrcGrad || e.src == kSrcGradOnly) {
        const int64_t at = (int64_t)i * ge.d + j;
        av = e.gtype == 0   ? static_cast<const float *>(e.a)[at]
             : e.gtype == 1 ? bf16_to_float(static_cast<const uint16_t *>(e.a)[at])
                            : f16_to_float(static_cast<const uint16_t *>(e.a)[at]);
    } else {
        av = static_cast<const float *>(e.a)[(int64_t)i * ge.ld + j];
    }
    if (e.src == kSrcGrad || e.src == kSrcDiff) av = fsub(av, e.b[(int64_t)i * ge.ld + j]);
    return av;
}

struct ExactLds {
    uint2 stage[4][kSub];      // the kept elements of a tile by owning wavefront
    uint32_t cnt[4];
    uint32_t zeros;
};

// The digits of Tc by counting over the whole vector.  All threads of the workgroup call this.
__device__ __forceinline__ uint64_t exact_threshold(const ExactSource &es, const TkGeom &ge, int i, ResolveLds &L)
{
    const int tid = threadIdx.x, nt = (int)blockDim.x;
    const uint32_t d = (uint32_t)ge.d;
    const SelKey sk = sel_key_of(ge.rand, ge.rand.step_now, i);
    int s_hi = 31 + ge.idx_bits;                                    // bits of comp still open
    uint64_t prefix = 0;
    uint32_t rank = ge.k;
    while (true) {
        const int s_lo = max(s_hi - kDigitBits, 0);
        const uint32_t mask = (1u << (s_hi - s_lo)) - 1u;
        for (int q = tid; q < kBins2; q += nt) L.lh[q] = 0;
        __syncthreads();
        for (int t = 0; t < ge.n_tiles; ++t) {
            for (int T = tid; T < kTile / 4; T += nt) {
                const uint32_t j0 = (uint32_t)t * kTile + 4u * (uint32_t)T;
                float x[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) x[c] = j0 + c < d ? exact_value(es, ge, i, j0 + c) : 0.f;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint64_t comp = composite(sel_key(sk, x[c], j0 + c), j0 + c, ge.idx_bits);
                    if (j0 + c < d && (comp >> s_hi) == prefix) atomicAdd(&L.lh[(uint32_t)(comp >> s_lo) & mask], 1u);
                }
            }
        }
        __syncthreads();
        find_rank_bin<kBins2>(L.lh, L.part, L.res, rank);          // rank <= elements under the prefix
        prefix = (prefix << (s_hi - s_lo)) | L.res[0];
        rank -= L.res[1];
        const uint32_t left = L.res[2];
        __syncthreads();
        if (s_lo == 0 || left == rank) return prefix << s_lo;      // last digit, or all under this prefix are kept
        s_hi = s_lo;
    }
}

// Lists the kept elements (comp >= tc) of the vector, tile by tile, as one run from the start of the worker's
// space, and writes every tile's record.  Coordinate 4 T + c of a tile (T = 0 .. 1023) belongs to the wavefront
// (T mod 256) / 64 of the listing pass.  All threads of the workgroup call this.
__device__ __forceinline__ void list_kept(const ExactSource &es, const TkGeom &ge, int i, uint64_t tc,
                                          uint2 *__restrict__ cand, uint4 *__restrict__ tile_dir, ExactLds &E)
{
    const int tid = threadIdx.x, nt = (int)blockDim.x;
    const int lane = tid & 63;
    const uint32_t d = (uint32_t)ge.d;
    const SelKey sk = sel_key_of(ge.rand, ge.rand.step_now, i);
    const bool skip_zeros = (es.src == kSrcStored && !sk.on);      // zeros are counted, not listed (as in tk_pass1)
    uint32_t run = 0;                                               // uniform over the workgroup
    if (tid < 4) E.cnt[tid] = 0;
    if (tid == 0) E.zeros = 0;
    __syncthreads();
    for (int t = 0; t < ge.n_tiles; ++t) {
        for (int T = tid; T < kTile / 4; T += nt) {                 // the same number of rounds for every thread
            const int owner = (T & (kThreads - 1)) >> 6;            // uniform over a wavefront
            const uint32_t j0 = (uint32_t)t * kTile + 4u * (uint32_t)T;
            float x[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = j0 + c < d ? exact_value(es, ge, i, j0 + c) : 0.f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t j = j0 + c;
                bool hit = j < d && composite(sel_key(sk, x[c], j), j, ge.idx_bits) >= tc;
                if (skip_zeros) {
                    const bool zero = j < d && mag_key(x[c]) == 0u;
                    const uint64_t zm = __ballot(zero);
                    if (lane == 0 && zm) atomicAdd(&E.zeros, (uint32_t)__popcll(zm));
                    hit = hit && !zero;
                }
                const uint64_t hm = __ballot(hit);
                uint32_t at = 0;
                if (lane == 0 && hm) at = atomicAdd(&E.cnt[owner], (uint32_t)__popcll(hm));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(hm & ((1ull << lane) - 1ull));
                if (hit) E.stage[owner][at] = make_uint2(j, __float_as_uint(x[c]));
            }
        }
        __syncthreads();
        const uint32_t cnt[4] = {E.cnt[0], E.cnt[1], E.cnt[2], E.cnt[3]};
        if (tid == 0)
            tile_dir[(int64_t)i * ge.n_tiles + t] = make_uint4(run, cnt[0] | (cnt[1] << 16), cnt[2] | (cnt[3] << 16), E.zeros);
        uint2 *dst = cand + worker_base(ge, i) + run;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            for (uint32_t q = tid; q < cnt[w]; q += nt) dst[q] = E.stage[w][q];
            dst += cnt[w];
        }
        run += cnt[0] + cnt[1] + cnt[2] + cnt[3];
        __syncthreads();
        if (tid < 4) E.cnt[tid] = 0;
        if (tid == 0) E.zeros = 0;
        __syncthreads();
    }
}

__device__ __forceinline__ uint64_t exact_select(const ExactSource &es, const TkGeom &ge, int i, uint2 *__restrict__ cand,
                                                 uint4 *__restrict__ tile_dir, ResolveLds &L, ExactLds &E)
{
    const uint64_t tc = exact_threshold(es, ge, i, L);
    list_kept(es, ge, i, tc, cand, tile_dir, E);
    return tc;
}

// xs: the stored rows under error feedback with magnitude keys (where zeros are counted instead of listed and
// the threshold may lie among them), else null.  es: how the compressed vector is re-formed, for a worker whose
// lists did not fit.
//
// Bound by latency: one workgroup per vector, and its instructions come from memory after every long pass.  The branches that
// a usual step does not take are marked, so that what it runs lies together (us, unmarked / marked, teams of 8 in both:
// n = 8, d = 110 M, k = 0.1 % 9.0 / 8.0, n = 16, d = 11.2 M, k = 1 % 7.9 / 7.1, Rand-k n = 16, d = 1.2 M 5.5 / 4.8).
__global__ __launch_bounds__(kResolveThreads) void tk_resolve(TkGeom ge, TkWorker *__restrict__ ws,
                                                              const uint64_t *__restrict__ dense,
                                                              const uint2 *__restrict__ dense_dir,
                                                              uint32_t *__restrict__ cursor,
                                                              uint32_t *__restrict__ cursor_b,
                                                              uint32_t *__restrict__ hist1,
                                                              uint32_t *__restrict__ histf,
                                                              uint32_t *__restrict__ hist_full,
                                                              uint32_t *__restrict__ hist2,
                                                              const uint32_t *__restrict__ piece_bits,
                                                              uint2 *__restrict__ cand, uint4 *__restrict__ tile_dir,
                                                              const float *__restrict__ xs, ExactSource es)
{
    __shared__ ResolveLds L;
    // the piece table of the usual path and the staging lists of exact_select are never needed together
    union Either {
        struct {
            uint32_t rpre[kMaxPieces + 1];
            uint32_t rstart[kMaxPieces];
            uint32_t plist[kFew];        // pieces that hold an element with the first digit of Tc
            uint32_t n_plist;
            uint64_t staged[kStaged];
        } pieces;
        ExactLds exact;
    };
    __shared__ Either U;
    uint32_t *rpre = U.pieces.rpre, *rstart = U.pieces.rstart;
    const int i = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    // what the usual case needs goes out before the record says whether it is the usual case
    const int pieces = ge.slices * ge.parts * 4;                 // a multiple of 4, at most 2 * kResolveThreads
    static_assert(kBinsFirst == kResolveThreads, "one bin of the first digit per thread");
    const uint32_t first_count = hist2[(int64_t)i * kBinsFirst + tid];
    uint4 two = make_uint4(0u, 0u, 0u, 0u);                      // {start, count} of pieces 2 tid and 2 tid + 1
    if (2 * tid < pieces) two = *reinterpret_cast<const uint4 *>(dense_dir + (int64_t)i * pieces + 2 * tid);
    const TkWorker w = ws[i];
    // Emptied for the next step: the cursors and candidate histograms (tk_compact was their last reader; zero already
    // in a step that did not use them) and the counts of the first digit.  slices <= 1024 threads.
    if (tid < ge.slices) cursor[(i * ge.slices + tid) * kCursorStride] = 0;
    for (int q = tid; q < kBins1; q += kResolveThreads) hist1[(int64_t)i * kBins1 + q] = 0;
    if (tid < kFineWindow) histf[(int64_t)i * kFineWindow + tid] = 0;
    hist2[(int64_t)i * kBinsFirst + tid] = 0;
    const int s_hi = (int)w.pshift + ge.idx_bits;
    uint64_t tc = (uint64_t)w.prefix << s_hi;
    const uint4 *dir_row = tile_dir + (int64_t)i * ge.n_tiles;
    if (__builtin_expect(w.overflow2 != 0u, 0)) {
        tc = exact_select(es, ge, i, cand, tile_dir, L, U.exact);
        if (tid == 0) ws[i].whole = kExact;          // for the records (comp_ams_get_selection_info)
    } else if (__builtin_expect(w.whole == kZeroTail, 0)) {
        tc = zero_tail_threshold(dir_row, xs + (int64_t)i * ge.ld, ge, w.rank, L);
    } else if (__builtin_expect(w.relisted && !w.whole, 0)) {
        // Lists made anew: the elements under the prefix stand in the worker's regions among those above it.  The first
        // digit is known as in the usual case; the elements under it are collected in LDS (one pass over the regions, a
        // region per wavefront) and searched there, or, where they are too many, found by digits over all regions.
        // First steps, us: CD-Adam n = 8, d = 11.2 M bf16 797 (1261 with every digit scanned over the regions), error
        // feedback n = 16, d = 11.2 M 929 (1026).
        L.lh[tid] = first_count;
        const int regions = ge.slices;
        uint32_t mine = 0;
        if (tid < regions) mine = min(cursor_b[(i * regions + tid) * kCursorStride], ge.region_cap);
        const uint32_t before = resolve_scan(mine, L.part, &L.res[3]);
        if (tid < regions) rpre[tid] = before;
        if (tid == regions - 1) rpre[regions] = before + mine;
        __syncthreads();
        const uint32_t cnt = rpre[regions];
        if (xs != nullptr && w.prefix == 0u && cnt < ge.k)
            // the bin of the smallest keys is listed without its zeros, so the lists hold every non-zero element:
            // fewer than k, and the k-th largest is a zero
            tc = zero_tail_threshold(dir_row, xs + (int64_t)i * ge.ld, ge, ge.k - cnt, L);
        else {
            const SelKey sk = sel_key_of(ge.rand, ge.rand.step_now, i);
            const uint2 *list = cand + worker_base(ge, i);
            find_rank_bin<kBinsFirst>(L.lh, L.part, L.res, w.rank);
            const int s_lo = s_hi - kFirstBits;
            const uint32_t left = L.res[2], rank1 = w.rank - L.res[1];
            const bool found = L.res[3] != 0u;
            const uint64_t prefix1 = ((uint64_t)w.prefix << kFirstBits) | L.res[0];
            if (found && left == rank1) {
                tc = prefix1 << s_lo;
            } else if (found && left <= (uint32_t)kStaged) {
                if (tid == 0) L.n_few = 0;
                __syncthreads();
                for (int reg = wave; reg < regions; reg += kResolveThreads / kWave) {
                    const uint32_t count = rpre[reg + 1] - rpre[reg];
                    const uint2 *src = list + (uint32_t)reg * ge.region_cap;
                    for (uint32_t q0 = 0; q0 < count; q0 += 8 * kWave) {
                        uint2 e[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const uint32_t q = q0 + u * kWave + lane;
                            e[u] = src[min(q, count - 1u)];
                        }
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const uint64_t comp = composite(sel_key(sk, __uint_as_float(e[u].y), e[u].x), e[u].x, ge.idx_bits);
                            if (q0 + u * kWave + lane < count && (comp >> s_lo) == prefix1) {
                                const uint32_t at = atomicAdd(&L.n_few, 1u);
                                if (at < (uint32_t)kStaged) U.pieces.staged[at] = comp;
                            }
                        }
                    }
                }
                __syncthreads();
                auto staged = [&](const uint32_t (&q)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
#pragma unroll
                    for (int u = 0; u < kScanUnroll; ++u) comp[u] = q[u] < left ? U.pieces.staged[q[u]] : 0ull;
                };
                tc = resolve_digits(staged, left, prefix1, rank1, s_lo, L);
            } else if (found) {
                int top = 1;
                while (2 * top < regions) top *= 2;
                auto fetch = [&](const uint32_t (&q)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
                    if (q[0] >= cnt) return;
                    int r[kScanUnroll];
                    uint32_t in[kScanUnroll];
#pragma unroll
                    for (int u = 0; u < kScanUnroll; ++u) {
                        r[u] = 0;
                        in[u] = min(q[u], cnt - 1u);
                    }
                    for (int bit = top; bit > 0; bit >>= 1) {
                        uint32_t start[kScanUnroll];
#pragma unroll
                        for (int u = 0; u < kScanUnroll; ++u) start[u] = rpre[min(r[u] + bit, regions)];
#pragma unroll
                        for (int u = 0; u < kScanUnroll; ++u) r[u] = (start[u] <= in[u] && r[u] + bit < regions) ? r[u] + bit : r[u];
                    }
                    uint2 e[kScanUnroll];
#pragma unroll
                    for (int u = 0; u < kScanUnroll; ++u)
                        e[u] = list[(uint32_t)r[u] * ge.region_cap + (in[u] - rpre[r[u]])];
#pragma unroll
                    for (int u = 0; u < kScanUnroll; ++u)
                        comp[u] = composite(sel_key(sk, __uint_as_float(e[u].y), e[u].x), e[u].x, ge.idx_bits);
                };
                tc = resolve_digits(fetch, cnt, prefix1, rank1, s_lo, L);
            }
        }
    } else if (__builtin_expect(!w.whole, 1)) {
        // tk_compact counted the first digit below the prefix while it copied: take its counts
        L.lh[tid] = first_count;
        const uint64_t *wdense = dense + region_base(ge, i, 0);
        // exclusive prefix sum of the piece counts, two pieces per thread
        const uint2 a = make_uint2(two.x, two.y), b = make_uint2(two.z, two.w);
        const uint32_t incl = wave_scan(a.y + b.y);
        if (lane == kWave - 1) L.part[wave] = incl;
        __syncthreads();
        const uint32_t before = waves_before(L.part, wave);
        const uint32_t excl = before + incl - (a.y + b.y);
        if (2 * tid < pieces) {
            rpre[2 * tid] = excl;
            rstart[2 * tid] = a.x;
        }
        if (2 * tid + 1 < pieces) {
            rpre[2 * tid + 1] = excl + a.y;
            rstart[2 * tid + 1] = b.x;
        }
        if (tid == kResolveThreads - 1) rpre[pieces] = before + incl;   // threads past the pieces add 0
        __syncthreads();
        const uint32_t cnt = rpre[pieces];
        // Elements q[u] of the worker's dense set, found through the prefix sums of the piece counts: the piece of
        // q is the last one that starts at or before it.  The searches of a batch advance together, one bit of the
        // piece number per round and without branches, so that a round's LDS reads are independent: one search
        // after the other leaves a scan waiting on kScanUnroll chains of dependent LDS reads per batch.
        int top = 1;
        while (2 * top < pieces) top *= 2;
        auto fetch = [&](const uint32_t (&q)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
            if (q[0] >= cnt) return;                       // nothing for this thread in the batch
            int r[kScanUnroll];
            uint32_t in[kScanUnroll];
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) {
                r[u] = 0;
                in[u] = min(q[u], cnt - 1u);               // no branch around the loads: see tk_hist
            }
            for (int bit = top; bit > 0; bit >>= 1) {
                uint32_t start[kScanUnroll];
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u) start[u] = rpre[min(r[u] + bit, pieces)];   // rpre[pieces] = cnt
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u) r[u] = (start[u] <= in[u] && r[u] + bit < pieces) ? r[u] + bit : r[u];
            }
            uint32_t at[kScanUnroll];
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) at[u] = rstart[r[u]] + (in[u] - rpre[r[u]]);
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) comp[u] = wdense[at[u]];
        };
        if (__builtin_expect(xs != nullptr && w.prefix == 0u && w.rank > cnt, 0))
            // the threshold bin is the one of the smallest keys and the k-th largest lies below its listed
            // (non-zero) elements: among the zeros
            tc = zero_tail_threshold(dir_row, xs + (int64_t)i * ge.ld, ge, w.rank - cnt, L);
        else {
            // The first digit below the prefix from tk_compact's counts.  Usually at most kFew elements carry it:
            // they sit in at most as many pieces, which the pieces' bitmaps name, so only those pieces are read
            // (a few hundred elements instead of the whole threshold bin) and the elements ranked directly.
            constexpr int kTeam = 16, kTeams = kResolveThreads / kTeam;
            const FirstDigit fd = first_digit(ge, w.pshift);
            find_rank_bin<kBinsFirst>(L.lh, L.part, L.res, w.rank);          // barriers since L.lh was filled
            const uint32_t digit = L.res[0], left = L.res[2], rank1 = w.rank - L.res[1];
            const bool found = L.res[3] != 0u;                                // always: rank <= elements under the prefix
            if (__builtin_expect(found && left == rank1, 0)) {
                tc = digit_edge(fd, w.prefix, digit);                         // all with this digit are kept
            } else if (__builtin_expect(found && left <= (uint32_t)min(kFew, kResolveThreads), 1)) {
                if (tid == 0) {
                    U.pieces.n_plist = 0;
                    L.n_few = 0;
                }
                __syncthreads();
                for (int p = tid; p < pieces; p += kResolveThreads) {
                    const uint32_t word = piece_bits[((int64_t)i * pieces + p) * kPieceWords + (digit >> 5)];
                    if ((word >> (digit & 31u)) & 1u) {
                        const uint32_t slot = atomicAdd(&U.pieces.n_plist, 1u);
                        if (slot < (uint32_t)kFew) U.pieces.plist[slot] = (uint32_t)p;     // always: see n_listed
                    }
                }
                __syncthreads();
                const uint32_t n_listed = min(U.pieces.n_plist, (uint32_t)kFew);   // <= left: each names an element
                // A piece per team of 16 lanes, four loads of a lane in flight: where few pieces are named they are read in one
                // round trip, and where many are (ties) the teams take them at once.  us, n = 8, d = 110 M without ties, and
                // n = 16, d = 11.2 M bf16: a piece per wavefront 8.4 and 13.9, teams of 8 with four loads 8.0 and 10.2, teams of 16
                // with one load 7.9 and 10.2, with four 7.4 and 10.5.
                for (uint32_t q = tid / kTeam; q < n_listed; q += kTeams) {
                    const uint32_t p = U.pieces.plist[q];
                    const uint32_t first = rstart[p], count = rpre[p + 1] - rpre[p];
                    for (uint32_t e = tid % kTeam; e < count; e += 4 * kTeam) {
                        uint64_t comp[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) comp[u] = wdense[first + min(e + u * kTeam, count - 1u)];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (e + u * kTeam < count && digit_of(fd, comp[u]) == digit) {
                                const uint32_t slot = atomicAdd(&L.n_few, 1u);
                                if (slot < (uint32_t)kFew) L.few[slot] = comp[u];
                            }
                        }
                    }
                }
                __syncthreads();
                tc = rank_few(left, rank1, L);
            } else if (found && left <= (uint32_t)kStaged) {
                // Many elements under the first digit, for instance ties by the hundred thousand.  The
                // elements are collected in LDS once, a piece per team of lanes and four pieces of a team in flight,
                // and the further digits scan LDS; through the piece table every digit was a scan of the whole bin.
                const int team = tid / kTeam, tl = tid % kTeam;
                if (tid == 0) L.n_few = 0;
                __syncthreads();
                auto collect = [&](uint64_t comp, bool valid) {
                    const bool hit = valid && digit_of(fd, comp) == digit;
                    const uint64_t hm = __ballot(hit);
                    if (!hm) return;
                    uint32_t at = 0;
                    if (lane == 0) at = atomicAdd(&L.n_few, (uint32_t)__popcll(hm));
                    at = __builtin_amdgcn_readfirstlane(at) + __popcll(hm & ((1ull << lane) - 1ull));
                    if (hit && at < (uint32_t)kStaged) U.pieces.staged[at] = comp;
                };
                for (int p0 = 0; p0 < pieces; p0 += 4 * kTeams) {              // uniform over the workgroup
                    uint32_t first[4], count[4], most = 0;
                    uint64_t comp[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int p = p0 + u * kTeams + team;
                        first[u] = p < pieces ? rstart[p] : 0u;
                        count[u] = p < pieces ? rpre[p + 1] - rpre[p] : 0u;
                        comp[u] = wdense[(uint32_t)tl < count[u] ? first[u] + tl : 0u];
                        most = max(most, count[u]);
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) collect(comp[u], (uint32_t)tl < count[u]);
                    for (uint32_t e = kTeam; __any(e < most); e += kTeam) {    // uniform over the wavefront
#pragma unroll
                        for (int u = 0; u < 4; ++u) comp[u] = wdense[e + tl < count[u] ? first[u] + e + tl : 0u];
#pragma unroll
                        for (int u = 0; u < 4; ++u) collect(comp[u], e + tl < count[u]);
                    }
                }
                __syncthreads();
                auto staged = [&](const uint32_t (&q)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
#pragma unroll
                    for (int u = 0; u < kScanUnroll; ++u) comp[u] = q[u] < left ? U.pieces.staged[q[u]] : 0ull;
                };
                const DigitBits known = digit_bits(fd, w.prefix, digit);
                // (a bin of the further digits may hold ties, which are not among the smallest other magnitudes)
                tc = resolve_digits<false>(staged, left, known.prefix, rank1, known.open, L);
            } else if (found) {
                const DigitBits known = digit_bits(fd, w.prefix, digit);
                tc = resolve_digits(fetch, cnt, known.prefix, rank1, known.open, L);
            }
        }
    }
    if (__builtin_expect(w.relisted != 0u, 0)) {               // tk_compact was the last reader of the full histogram
        if (tid < ge.slices) cursor_b[(i * ge.slices + tid) * kCursorStride] = 0;
        for (int q = tid; q < kBins1; q += kResolveThreads) hist_full[(int64_t)i * kBins1 + q] = 0;
    }
    if (tid == 0) {
        // Tc = 0 keeps every coordinate.  Below k = d it is the lower edge of a bin of the smallest keys whose listed elements
        // are all kept: zeros, which are not listed then (xs), must stay out.
        if (xs != nullptr && tc == 0 && ge.k < ge.d) tc = 1ull << ge.idx_bits;
        finish_worker(ws, i, w, tc, ge, w.relisted != 0);
    }
}


// ---------------------------------------------------------------------------------------------
// The selection in one launch: short vectors (at most kSmallTiles tiles), and longer ones whose lists one workgroup
// holds (one_launch_select).
// On such a vector every kernel of the selection chain is a launch on an idle chip, and three of them cost more
// than the work.  The listing pass is tk_pass1 itself, on a short vector with a single candidate region per vector (few tiles share
// its cursor); then one workgroup per vector finds the threshold from the list by itself - the digits of Tc over
// the listed comp values, after listing the vector again when the list does not hold the k-th largest.  The tile directory and the list have the
// usual form, so the kernels after it and the getters follow unchanged.  (Finding the threshold inside the listing
// pass, by the workgroup that finishes a worker's last tile, was built and measured: the device-scope fences it needs
// on this multi-XCD part cost more than the launch they save - 21.6 us against 6 + 5.)
// Bound by latency: a list of up to kScanUnroll entries per thread (a vector of 65 536 coordinates lists 1.2 k) is read
// once, into registers, and the digits are found from those.
// The first digit is the fine bin, counted from the guess's, so that a few entries are left to rank.  (With the top 12 bits of comp,
// 6 % wide, up to 256 were left, and ranking those against each other took 3.5 us of 9.3.  Kernel, and step plus get_theta, us, that
// / this, with the scans by lane permutes as well: error feedback n = 4, d = 65 536, k = 1 % 10.4 / 6.8, 33.9 / 29.3, n = 8,
// d = 20 000, k = 2 % 9.1 / 5.6, 34.5 / 30.3; naive n = 8, d = 40 000, k = 5 % bf16 8.0 / 5.6, 32.9 / 29.2.)
constexpr int kSmallTiles = 16;
constexpr int kShortFine = 2048;  // fine bins of the first digit: four octaves above the guess

// After a miss (a guess that was too high, a full region, the first step of a vector of few tiles) the workgroup lists the
// vector again by itself: one pass counts the coarse bins, a second lists what lies in the k-th largest's bin or above,
// kShortBatch tiles in flight.  Bound by one compute unit's loads and LDS atomics.  Counting the whole composite key over
// the vector at once (exact_select: up to six sweeps of scalar loads, one more to list) made one miss cost what ten steps
// gain.  Step plus get_theta, n = 8, d = 65 536, k = 1 %, scale a thousandth for 6 steps of 12, us, the three launches of long
// vectors / exact_select at every miss / this: naive 46.8 / 48.1 / 36.9, CD-Adam 74.4 / 129.0 / 67.8; fresh gradients, n = 32,
// d = 60 000: naive 55.0 / 59.0 / 45.2, error feedback (which had exact_select before) 69.6 / 65.9 / 52.5.
constexpr int kShortBatch = 4;
static_assert((int64_t)kShortBatch * kTile >= (int64_t)1 << kTieBits, "digit_of: longer vectors have at least kTieBits index bits");
constexpr int kRankAll = 128;     // a list of at most this many entries is ranked as it is, without digits (Rand-k under error
                                  // feedback, n = 8, d = 5000, k = 50: 34.3 -> 32.2 us; at 200 to 256 entries digits are
                                  // faster, d = 20 000, k = 200: 33.9 ranked, 33.5)
static_assert(kRankAll <= kFew, "held in ResolveLds::few");
struct ShortLds {
    uint32_t count[kWave], zeros[kShortBatch];
};
// What is known of Tc: the bits of comp above the `open` low ones, and its rank among the elements that carry them.
struct ShortDigits {
    uint64_t prefix;
    uint32_t rank;
    int open;
};
static_assert(kTile == 4 * kResolveThreads, "a float4 of each tile per thread");
static_assert(kShortBatch * kResolveThreads / kWave == kWave, "a wavefront's count of a tile per lane");

// Lists the vector again, as one run from the start of its space, and writes every tile's record.  Returns the number of
// entries, or kNoSpace where they do not fit (the list is then of no use).  All kResolveThreads threads call this; ends
// with a barrier.
template <int kSrc, typename G>
__device__ __forceinline__ uint32_t list_short_again(const TkGeom &ge, int i, const void *__restrict__ a,
                                                     const float *__restrict__ b, const SelKey &sk,
                                                     uint2 *__restrict__ cand, uint4 *__restrict__ tile_dir, ResolveLds &L,
                                                     ShortLds &S, ShortDigits &top)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t d = (uint32_t)ge.d;
    const float *brow = (kSrc == kSrcGrad || kSrc == kSrcDiff) ? b + (int64_t)i * ge.ld : nullptr;
    const bool skip_zeros = kSrc == kSrcStored && !sk.on;               // zeros are counted, not listed (as in tk_pass1)
    for (int q = tid; q < kBins1; q += kResolveThreads) L.lh[q] = 0;
    __syncthreads();
    for (int t0 = 0; t0 < ge.n_tiles; t0 += kShortBatch) {
        Source4<kSrc, G> v[kShortBatch];
#pragma unroll
        for (int u = 0; u < kShortBatch; ++u)
            if (t0 + u < ge.n_tiles) v[u].load(a, i, ge, brow, (uint32_t)(t0 + u) * kTile + 4 * tid, d);
#pragma unroll
        for (int u = 0; u < kShortBatch; ++u) {
            if (t0 + u >= ge.n_tiles) continue;
            const float4 v4 = v[u].value();
            const float x[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t j = (uint32_t)(t0 + u) * kTile + 4 * tid + c;
                const uint32_t bin = sel_key(sk, x[c], j) >> kShift1;
                if (bin != 0 && j < d) atomicAdd(&L.lh[bin], 1u);      // bin 0 is the remainder
            }
        }
    }
    __syncthreads();
    find_rank_bin<kBins1>(L.lh, L.part, L.res, ge.k);
    const uint32_t prefix = L.res[3] ? L.res[0] : 0u;                   // fewer than k counted: bin 0
    if (L.res[3]) top = {prefix, ge.k - L.res[1], kShift1 + ge.idx_bits};
    uint32_t run = 0;
    for (int t0 = 0; t0 < ge.n_tiles; t0 += kShortBatch) {              // uniform over the workgroup
        float x[kShortBatch][4];
        uint32_t hits = 0, count[kShortBatch];
        Source4<kSrc, G> s[kShortBatch] = {};
#pragma unroll
        for (int u = 0; u < kShortBatch; ++u)
            if (t0 + u < ge.n_tiles) s[u].load(a, i, ge, brow, (uint32_t)(t0 + u) * kTile + 4 * tid, d);
#pragma unroll
        for (int u = 0; u < kShortBatch; ++u) {
            const float4 v = s[u].value();
            x[u][0] = v.x;
            x[u][1] = v.y;
            x[u][2] = v.z;
            x[u][3] = v.w;
        }
        if (tid < kShortBatch) S.zeros[tid] = 0;                         // read, in the round before, by these threads' wavefront
        __syncthreads();                                                // and the counts by all
#pragma unroll
        for (int u = 0; u < kShortBatch; ++u) {
            uint32_t zeros = 0;
            count[u] = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t j = (uint32_t)(t0 + u) * kTile + 4 * tid + c;        // at or beyond d in tiles past the last
                bool hit = j < d && (sel_key(sk, x[u][c], j) >> kShift1) >= prefix;
                if (skip_zeros) {
                    const bool zero = j < d && mag_key(x[u][c]) == 0u;
                    zeros += (uint32_t)__popcll(__ballot(zero));
                    hit = hit && !zero;
                }
                count[u] += (uint32_t)__popcll(__ballot(hit));
                hits |= (hit ? 1u : 0u) << (u * 4 + c);
            }
            if (lane == 0) {
                // in the order of the list: tile by tile, the listing pass's wavefronts one after the other (wavefront
                // wave & 3 of it owns what this one holds, its row wave >> 2)
                S.count[u * 16 + (wave & 3) * 4 + (wave >> 2)] = count[u];
                if (zeros) atomicAdd(&S.zeros[u], zeros);
            }
        }
        __syncthreads();
        // every wavefront adds the counts up for itself
        const uint32_t mine = S.count[lane], incl = wave_scan(mine), total = scan_total(incl);
        if (total > ge.region_cap - run) return kNoSpace;               // uniform over the workgroup
        if (wave == 0) {
            // lane 16 u + 4 w: the first of the four counts of wavefront w of tile t0 + u
            uint32_t quad = mine + (uint32_t)__shfl_down((int)mine, 1, kWave);
            quad += (uint32_t)__shfl_down((int)quad, 2, kWave);
            const uint32_t w1 = (uint32_t)__shfl_down((int)quad, 4, kWave), w2 = (uint32_t)__shfl_down((int)quad, 8, kWave),
                           w3 = (uint32_t)__shfl_down((int)quad, 12, kWave);
            if ((lane & 15) == 0 && t0 + (lane >> 4) < ge.n_tiles)
                tile_dir[(int64_t)i * ge.n_tiles + t0 + (lane >> 4)] =
                    make_uint4(run + incl - mine, quad | (w1 << 16), w2 | (w3 << 16), S.zeros[lane >> 4]);
        }
        uint2 *dst = cand + worker_base(ge, i) + run;
#pragma unroll
        for (int u = 0; u < kShortBatch; ++u) {
            uint32_t at = (uint32_t)__shfl((int)(incl - mine), u * 16 + (wave & 3) * 4 + (wave >> 2), kWave);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const bool hit = (hits >> (u * 4 + c)) & 1u;
                const uint32_t slot = wave_append(hit, at);
                if (hit) dst[slot] = make_uint2((uint32_t)(t0 + u) * kTile + 4 * tid + c, __float_as_uint(x[u][c]));
            }
        }
        run += total;
    }
    __syncthreads();                                                    // the list is read back by other threads
    return run;
}

// The k-th largest comp value of a list that lies in the regions of vector i (lane q holds the count `mine` of region q, `total` in
// all, at least k), every element at or above the guess's fine bin.  A wavefront holds the entries of two or four regions in
// registers, all loads in flight at once, and the first digit is the fine bin above the guess (see tk_small_select).  Many entries
// in the threshold's bin, or a threshold beyond the bins, are searched by digits through the regions' prefix sums.  top: what the
// first digit tells.  Bound by one round trip for the entries and their LDS atomics.
constexpr int kHeldRegions = 32, kHeldPerLane = 24;
static_assert(kHeldPerLane * kResolveThreads == kHeldEntries, "launch_rules.h");
__device__ __forceinline__ uint64_t select_in_regions(const TkGeom &ge, int i, const uint2 *__restrict__ list, uint32_t mine,
                                                      uint32_t total, uint32_t guess, const SelKey &sk, uint32_t *rpre,
                                                      ResolveLds &L, ShortDigits &top)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool four = ge.slices > kHeldRegions;                          // regions of a wavefront: four or two
    const int open = kFineShift + ge.idx_bits;
    uint2 e[kHeldPerLane];
    uint32_t held = 0;                                                   // bit u: e[u] is an entry
#pragma unroll
    for (int u = 0; u < kHeldPerLane; ++u) {
        const int region = four ? 4 * wave + u / (kHeldPerLane / 4) : 2 * wave + u / (kHeldPerLane / 2);
        const uint32_t at = (four ? u % (kHeldPerLane / 4) : u % (kHeldPerLane / 2)) * kWave + lane;
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)mine, region);
        held |= (at < cnt ? 1u : 0u) << u;
        e[u] = list[(uint32_t)region * ge.region_cap + (at < cnt ? at : 0u)];       // no branch around the load
    }
    auto bin_of = [&](const uint2 &c) {
        return min((sel_key(sk, __uint_as_float(c.y), c.x) >> kFineShift) - guess, (uint32_t)kShortFine - 1u);
    };
    // entries of the wavefront's regions beyond those held (uneven lists)
    auto others = [&](auto &&f) {
        const int regions = four ? 4 : 2;
        for (int r = regions * wave; r < regions * (wave + 1); ++r) {
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)mine, r);
            for (uint32_t at = kHeldPerLane * kWave / regions + lane; at < cnt; at += kWave) f(list[(uint32_t)r * ge.region_cap + at]);
        }
    };
    uint32_t bins[kHeldPerLane];
#pragma unroll
    for (int u = 0; u < kHeldPerLane; ++u) {
        bins[u] = bin_of(e[u]);
        if ((held >> u) & 1u) atomicAdd(&L.lh[bins[u]], 1u);
    }
    others([&](const uint2 &c) { atomicAdd(&L.lh[bin_of(c)], 1u); });
    __syncthreads();
    find_rank_bin<kShortFine>(L.lh, L.part, L.res, ge.k);
    const uint32_t bin = L.res[0], left = L.res[2], rank = ge.k - L.res[1];
    if (bin != (uint32_t)kShortFine - 1u) {                              // the last one holds all beyond as well
        top = {guess + bin, rank, open};
        if (left <= (uint32_t)kFew) {
            auto take = [&](const uint2 &c) {
                L.few[atomicAdd(&L.n_few, 1u)] = composite(sel_key(sk, __uint_as_float(c.y), c.x), c.x, ge.idx_bits);
            };
#pragma unroll
            for (int u = 0; u < kHeldPerLane; ++u)
                if (((held >> u) & 1u) && bins[u] == bin) take(e[u]);
            others([&](const uint2 &c) {
                if (bin_of(c) == bin) take(c);
            });
            __syncthreads();
            return rank_few(left, rank, L);
        }
    }
    const uint32_t before = wave_scan(mine) - mine;
    if (tid < ge.slices) rpre[tid] = before;
    if (tid == 0) rpre[ge.slices] = total;
    __syncthreads();
    auto fetch = [&](const uint32_t (&q)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
        if (q[0] >= total) return;
        int r[kScanUnroll];
        uint32_t in[kScanUnroll];
#pragma unroll
        for (int u = 0; u < kScanUnroll; ++u) {
            r[u] = 0;
            in[u] = min(q[u], total - 1u);
        }
        for (int bit = ge.slices / 2; bit > 0; bit >>= 1) {
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) r[u] = rpre[r[u] + bit] <= in[u] ? r[u] + bit : r[u];
        }
        uint2 c[kScanUnroll];
#pragma unroll
        for (int u = 0; u < kScanUnroll; ++u) c[u] = list[(uint32_t)r[u] * ge.region_cap + (in[u] - rpre[r[u]])];
#pragma unroll
        for (int u = 0; u < kScanUnroll; ++u) comp[u] = composite(sel_key(sk, __uint_as_float(c[u].y), c[u].x), c[u].x, ge.idx_bits);
    };
    return resolve_digits<false>(fetch, total, top.prefix, top.rank, top.open, L);
}

// ge: the geometry the vectors were listed with, and so `count`: the regions' cursors, kCursorStride words apart (cleared here for
// the next step).  kRegions: kHeldRegions regions or twice as many (lists of up to kHeldEntries entries, see one_launch_select);
// else a single one per vector (short vectors).  a, b: how a vector is re-formed (Source4).  A vector that was listed again
// raises the handle's flag (kRegions; see flag_record), which only the host's next choice of launches depends on.
template <int kSrc, typename G, bool kRegions>
__global__ __launch_bounds__(kResolveThreads) void tk_small_select(TkGeom ge, TkWorker *__restrict__ ws,
                                                                   uint2 *__restrict__ cand, uint32_t *__restrict__ count,
                                                                   uint4 *__restrict__ tile_dir, const void *__restrict__ a,
                                                                   const float *__restrict__ b)
{
    __shared__ ResolveLds L;
    __shared__ union {
        ShortLds again;
        ExactLds exact;
    } U;
    __shared__ uint32_t rpre[kRegions ? kWave + 1 : 1];
    const int i = blockIdx.x;
    const int tid = threadIdx.x;
    TkGeom sge = ge;                 // a vector's whole space as one region, which it becomes where it is listed again
    sge.region_cap = (uint32_t)ge.slices * ge.region_cap;
    sge.slices = 1;
    const uint2 *list = cand + worker_base(sge, i);
    uint32_t total, mine = 0;        // kRegions: lane q's own region holds `mine`
    if constexpr (kRegions) {
        if ((tid & 63) < ge.slices) mine = count[(i * ge.slices + (tid & 63)) * kCursorStride];
        total = scan_total(wave_scan(mine));
    } else {
        total = count[i * kCursorStride];
    }
    const TkWorker w = ws[i];
    for (int q = tid; q < kShortFine; q += kResolveThreads) L.lh[q] = 0;
    if (tid == 0) L.n_few = 0;
    __syncthreads();                                                  // nothing waits for memory yet
    const SelKey sk = sel_key_of(sge.rand, sge.rand.step_now, i);
    const bool zeros_listed = kSrc != kSrcStored || sk.on;           // see tk_pass1
    const ExactSource es{kSrc, std::is_same<G, float>::value ? 0 : std::is_same<G, uint16_t>::value ? 1 : 2, a, b};
    // a list of every non-zero element (the guess was 0) needs no other, however short it is
    const bool missed = w.overflow || (total < sge.k && (zeros_listed || w.guess != 0u));
    ShortDigits top = {0ull, sge.k, 31 + sge.idx_bits};
    // rare only where a flag is raised: short vectors gain nothing by the hint (CD-Adam n = 4, d = 16 908 39.2 us with it, 38.8 without)
    if (kRegions ? __builtin_expect(missed, 0) : missed)
        total = list_short_again<kSrc, G>(sge, i, a, b, sk, cand, tile_dir, L, U.again, top);
    uint64_t tc;
    if (missed && total == kNoSpace) {
        tc = exact_select(es, sge, i, cand, tile_dir, L, U.exact);
    } else if (kRegions && !missed && total >= sge.k) {
        tc = select_in_regions(ge, i, list, mine, total, w.guess, sk, rpre, L, top);
    } else if (total >= sge.k) {
        // every element at or above the guess is listed and there are at least k: Tc is the k-th largest of the
        // list (the comp value itself: a digit's bin may reach below the guess, where nothing is listed)
        auto comp_of = [&](uint32_t q) -> uint64_t {
            if (q >= total) return 0ull;
            const uint2 e = list[q];
            return composite(sel_key(sk, __uint_as_float(e.y), e.x), e.x, sge.idx_bits);
        };
        if (total <= (uint32_t)kRankAll) {
            if ((uint32_t)tid < total) L.few[tid] = comp_of(tid);
            __syncthreads();
            tc = rank_few(total, sge.k, L);
        } else if (total <= (uint32_t)(kScanUnroll * kResolveThreads)) {
            uint64_t held[kScanUnroll];
#pragma unroll
            for (int u = 0; u < kScanUnroll; ++u) held[u] = comp_of(u * kResolveThreads + tid);
            auto fetch = [&](const uint32_t (&)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u) comp[u] = held[u];       // one batch: q[u] = u * kResolveThreads + tid
            };
            // The first digit: the fine bin, counted from the guess's, below which nothing is listed, up to kShortFine bins.
            // The threshold lies a little above the guess, so its bin is among them and holds a few entries.
            bool found = false;
            if (!missed) {
                const uint32_t guess = w.guess;
                const int open = kFineShift + sge.idx_bits;
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u)
                    if (u * kResolveThreads + tid < total)
                        atomicAdd(&L.lh[min((uint32_t)(held[u] >> open) - guess, (uint32_t)kShortFine - 1u)], 1u);
                __syncthreads();
                find_rank_bin<kShortFine>(L.lh, L.part, L.res, sge.k);
                const uint32_t bin = L.res[0], left = L.res[2];
                top = {guess + bin, sge.k - L.res[1], open};
                if (bin == (uint32_t)kShortFine - 1u) {                          // holds all beyond as well
                    top = {0ull, sge.k, 31 + sge.idx_bits};
                } else if (left <= (uint32_t)kFew) {
#pragma unroll
                    for (int u = 0; u < kScanUnroll; ++u)
                        if (u * kResolveThreads + tid < total && (held[u] >> open) == top.prefix)
                            L.few[atomicAdd(&L.n_few, 1u)] = held[u];
                    __syncthreads();
                    tc = rank_few(left, top.rank, L);
                    found = true;
                }
            }
            if (!found) tc = resolve_digits<false>(fetch, total, top.prefix, top.rank, top.open, L);
        } else {
            auto fetch = [&](const uint32_t (&q)[kScanUnroll], uint64_t (&comp)[kScanUnroll]) {
#pragma unroll
                for (int u = 0; u < kScanUnroll; ++u) comp[u] = comp_of(q[u]);
            };
            tc = resolve_digits<false>(fetch, total, top.prefix, top.rank, top.open, L);
        }
    } else {
        // every non-zero element is listed and they are fewer than k: the threshold lies among the zeros, which the
        // list leaves out - all candidates are kept, and Tc comes from counting over the vector (a long one: from the tiles' counts)
        if constexpr (kRegions)
            tc = zero_tail_threshold(tile_dir + (int64_t)i * ge.n_tiles, static_cast<const float *>(a) + (int64_t)i * ge.ld, ge,
                                     ge.k - total, L);
        else
            tc = exact_threshold(es, sge, i, L);
    }
    if (kRegions && tid < ge.slices) count[(i * ge.slices + tid) * kCursorStride] = 0;
    if (tid == 0) {
        if (kRegions && missed) raise_flag(ws[ge.n]);
        ws[i].relisted = missed ? 1u : 0u;
        ws[i].whole = missed && total == kNoSpace ? kExact : 0u;
        if (kRegions) {                                                // for the records, as tk_compact leaves them
            ws[i].prefix = (uint32_t)top.prefix;
            ws[i].pshift = (uint32_t)(top.open - ge.idx_bits);
            ws[i].rank = top.rank;
        }
        finish_worker(ws, i, w, tc, sge, missed);
        if (!kRegions) count[i * kCursorStride] = 0;
    }
}

// CD-Adam (Algorithm 1): selection buffers of the server's own Top-k - the same structures as the
// workers', for a single vector.
struct TkSide {
    TkGeom ge;                 // n = 1
    TkWorker *ws;
    uint2 *cand;
    uint32_t *cursor;
    uint4 *tile_dir;
};

// Per tile: ghat_i += c_i (line 6), ghat += mean of the c_i (line 8), and the server's vector w = ghat - gtilde (line 9), whose
// candidates are listed straight from the registers; sv: the server's selection.  The scattered additions are most of it on long
// rows, each the read and the write of a whole line in memory (n = 8, d = 11.2 M, 1.4 M kept values: 51 of 77 us); the listing here
// saves a launch that read ghat and gtilde again (two kernels / one, us: the same bf16 94.8 / 91.4, d = 2 M 17.5 / 14.4, step plus
// get_theta 342 / 334 and 112 / 104).  kEarly: ghat and gtilde are loaded first, see merge_loads_early.
template <int kKey, bool kEarly>
__global__ __launch_bounds__(kThreads) void tk_merge(TkGeom ge, const TkWorker *__restrict__ ws,
                                                     const uint2 *__restrict__ cand,
                                                     const uint4 *__restrict__ tile_dir,
                                                     float *__restrict__ ghat_rows, float *__restrict__ ghat,
                                                     const float *__restrict__ gtil, float n_workers, TkSide sv)
{
    __shared__ float acc[kTile];
    __shared__ uint32_t sh[9];
    const int t = blockIdx.x;
    const uint32_t base = (uint32_t)t * kTile, d = (uint32_t)ge.d;
    const int tid = threadIdx.x;
    float4 gh[4], gt[4];
    auto load_server = [&] {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            gh[r] = ld4(ghat + base + 4 * (tid + kThreads * r));
            gt[r] = ld4(gtil + base + 4 * (tid + kThreads * r));
        }
    };
    if (kEarly) load_server();
#pragma unroll
    for (int r = 0; r < 4; ++r) st4(acc + 4 * (tid + kThreads * r), make_float4(0.f, 0.f, 0.f, 0.f));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    sum_kept_tile<true>(acc, ge, ws, cand, tile_dir, t, ghat_rows, tid >> 6);
    if (!kEarly) load_server();
    float w[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = 4 * (tid + kThreads * r);
        const float4 a = ld4(acc + l);
        // padding coordinates: 0 + 0 / n; ghat moves only where some worker kept a coordinate
        const float4 nh = make_float4(fadd(gh[r].x, fdiv(a.x, n_workers)), fadd(gh[r].y, fdiv(a.y, n_workers)),
                                      fadd(gh[r].z, fdiv(a.z, n_workers)), fadd(gh[r].w, fdiv(a.w, n_workers)));
        st4_if_changed<false>(ghat + base + l, nh, gh[r]);
        w[r][0] = fsub(nh.x, gt[r].x);
        w[r][1] = fsub(nh.y, gt[r].y);
        w[r][2] = fsub(nh.z, gt[r].z);
        w[r][3] = fsub(nh.w, gt[r].w);
    }
    SelKey sk = sel_key_of(sv.ge.rand, sv.ge.rand.step_now, 0);
    sk.on = kKey == kKeyScore ? 1u : 0u;
    const uint32_t guess = sv.ws[0].guess;
    if (base + kTile <= d)
        list_registers<true, false>(w, base, d, guess, sk, sh, sv.ge, 0, t, sv.cand, sv.cursor, sv.tile_dir, &sv.ws[0].overflow);
    else
        list_registers<false, false>(w, base, d, guess, sk, sh, sv.ge, 0, t, sv.cand, sv.cursor, sv.tile_dir, &sv.ws[0].overflow);
}

// CD-Adam (Algorithm 1), lines 10 and 12-16: gtilde += c, c = the kept coordinates of w, then the
// AMSGrad update with gtilde.  Per tile; each wavefront handles its own coordinates.
template <bool kStreamState>
__global__ __launch_bounds__(kThreads) void tk_apply(TkSide sv, float *__restrict__ gtil, float *__restrict__ theta,
                                                     float *__restrict__ m, float *__restrict__ v,
                                                     float *__restrict__ vhat, AmsParams p)
{
    __shared__ float acc[kTile];
    const int t = blockIdx.x;
    const int64_t base = (int64_t)t * kTile;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int r = 0; r < 4; ++r) st4(acc + 4 * (tid + kThreads * r), make_float4(0.f, 0.f, 0.f, 0.f));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    {
        const uint4 rec = sv.tile_dir[t];
        const uint32_t c[4] = {rec.y & 0xffffu, rec.y >> 16, rec.z & 0xffffu, rec.z >> 16};
        uint32_t start = rec.x;
        for (int q = 0; q < wave; ++q) start += c[q];
        const uint64_t tc = sv.ws[0].tc;
        const SelKey sk = sel_key_of(sv.ge.rand, sv.ws[0].step_word, 0);
        const uint2 *src = sv.cand + start;          // a single vector: its space starts the array
        for (uint32_t q = lane; q < c[wave]; q += kWave) {
            const uint2 e = src[q];
            const float x = __uint_as_float(e.y);
            if (composite(sel_key(sk, x, e.x), e.x, sv.ge.idx_bits) >= tc) acc[e.x - (uint32_t)base] = x;   // distinct coordinates
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
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
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int l = 4 * (tid + kThreads * r);
        const int64_t j = base + l;
        const float4 c4 = ld4(acc + l);
        // c is +0 where nothing was kept; gtilde + 0 = gtilde
        const float4 g4 = make_float4(fadd(gt[r].x, c4.x), fadd(gt[r].y, c4.y), fadd(gt[r].z, c4.z),
                                      fadd(gt[r].w, c4.w));
        amsgrad_update4(th[r], mm[r], vv[r], vh[r], g4, p);
        st4_if_changed<kStreamState>(gtil + j, g4, gt[r]);      // gtilde moves at the k kept coordinates only
        st4_state<kStreamState>(theta + j, th[r]);
        st4_state<kStreamState>(m + j, mm[r]);
        st4_state<kStreamState>(v + j, vv[r]);
        st4_state<kStreamState>(vhat + j, vh[r]);
    }
}

// Getter support -------------------------------------------------------------------------------

// e_i of one worker in its defined form, from the stored x and the pending threshold.
__global__ __launch_bounds__(kThreads) void tk_materialize_error(const float *xrow, TkGeom ge, int worker,
                                                                 const TkWorker *__restrict__ w, float *out)
{
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= ge.d) return;
    const float x = xrow[j];
    const SelKey sk = sel_key_of(ge.rand, w->step_word, worker);
    out[j] = was_kept(kept_test(w->tc, ge.idx_bits), sel_key(sk, x, (uint32_t)j), (uint32_t)j) ? 0.f : x;
}

// The kept (index, value) pairs of one worker, in no particular order: candidates with
// comp >= Tc.  *count must be 0 on entry and ends at k.  One workgroup per tile; one atomic add
// per wavefront that found something.
__global__ __launch_bounds__(kThreads) void tk_gather_selected(TkGeom ge, int worker,
                                                               const TkWorker *__restrict__ ws,
                                                               const uint2 *__restrict__ cand,
                                                               const uint4 *__restrict__ tile_dir,
                                                               uint32_t *__restrict__ count,
                                                               uint32_t *__restrict__ out_idx,
                                                               float *__restrict__ out_val)
{
    const int lane = threadIdx.x & 63;
    const int t = blockIdx.x;
    const uint64_t tc = ws[worker].tc;
    const SelKey sk = sel_key_of(ge.rand, ws[worker].step_word, worker);
    const uint4 rec = tile_dir[(int64_t)worker * ge.n_tiles + t];
    const uint2 *src = cand + worker_base(ge, worker) + rec.x;
    const uint32_t total = (rec.y & 0xffffu) + (rec.y >> 16) + (rec.z & 0xffffu) + (rec.z >> 16);
    for (uint32_t q0 = 0; q0 < total; q0 += kThreads) {      // uniform over the workgroup
        const uint32_t q = q0 + threadIdx.x;
        uint2 c = make_uint2(0u, 0u);
        bool keep = false;
        if (q < total) {
            c = src[q];
            keep = composite(sel_key(sk, __uint_as_float(c.y), c.x), c.x, ge.idx_bits) >= tc;
        }
        const uint64_t km = __ballot(keep);
        if (km) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(count, (uint32_t)__popcll(km));
            at = __shfl(at, 0, kWave) + __popcll(km & ((1ull << lane) - 1ull));
            if (keep && at < ge.k) {
                out_idx[at] = c.x;
                out_val[at] = __uint_as_float(c.y);
            }
        }
    }
}

// The kept zeros of one worker's stored row when the threshold lies among them (key part of Tc is 0): the
// zeros at indices up to Tc's, appended to the pairs tk_gather_selected has written.
__global__ __launch_bounds__(kThreads) void tk_gather_zero_tail(const float *__restrict__ xrow, TkGeom ge,
                                                                const TkWorker *__restrict__ w,
                                                                uint32_t *__restrict__ count,
                                                                uint32_t *__restrict__ out_idx,
                                                                float *__restrict__ out_val)
{
    const KeptTest kt = kept_test(w->tc, ge.idx_bits);
    if (kt.tkey != 0u) return;
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool keep = j < ge.d && j <= (int64_t)kt.tj && mag_key(xrow[min(j, ge.d - 1)]) == 0u;
    const uint64_t km = __ballot(keep);
    if (km) {
        const int lane = threadIdx.x & 63;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(count, (uint32_t)__popcll(km));
        at = __shfl(at, 0, kWave) + __popcll(km & ((1ull << lane) - 1ull));
        if (keep && at < ge.k) {
            out_idx[at] = (uint32_t)j;
            out_val[at] = xrow[j];
        }
    }
}

// Wire form of a sparse message: (index, value bits) pairs.
__global__ __launch_bounds__(kThreads) void tk_pack_pairs(const uint32_t *__restrict__ idx, const float *__restrict__ val,
                                                          uint32_t k, uint2 *__restrict__ out)
{
    const uint32_t r = blockIdx.x * kThreads + threadIdx.x;
    if (r < k) out[r] = make_uint2(idx[r], __float_as_uint(val[r]));
}

}  // namespace cams
