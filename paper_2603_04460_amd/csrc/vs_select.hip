// Budget rule and TopK (Sec. "Adaptive Sparse Index Selection": k_d is the fewest top-ranked scores
// whose mass reaches tau_d, I_d = TopK(A_d, k_d)).
//
// Non-negative fp32 scores order like their bit patterns, so the k-th ranked score is found by a most-significant-digit radix
// descent.  A bucket of a pass carries ONE 64-bit weight: the INTEGER mass floor(score * 2^40), or the element count for the fixed
// budget and for the capacity.  Integer weights make every partial sum exact and independent of the order, so the threshold
// crossing is the same however the work is split.  Ties at the crossing value are taken in ascending index order.  The selected set,
// united with the forced leading indices, is then written in ascending order from ballots and counts (no atomics on the output path).
//
// Bound by latency: a few dependent steps, each a round trip to memory or a barrier, and by the instructions of 16 wavefronts on
// one compute unit, so one wavefront does the scans and the others wait for it.
//
// Short problems: one workgroup per (head, direction), select_kernel.  The first digit is cut where the scores are, keys >> 19 (16 buckets
// per octave up to 1.9375, everything above in the last one): its crossing bucket usually holds less than a percent of the scores.
// Those, the candidates, are put aside in index order and the remaining digits (10 bits each) only look at them.  Up to 8192 scores stay
// in registers, candidates in LDS.
// Long ones with a workspace: one workgroup per chunk of a problem (8192 scores up to 131072) and, after one kernel that clears, four: the histogram of
// the first digit, that of the second in the first's crossing bucket, both added to the problem's in the workspace with integer atomics; the chunk's
// counts of the last digit in the second's crossing bucket; the crossing value, from the counts of all chunks, and the emission.  Every pass looks at
// a chunk's own scores only, however they crowd.  A problem whose selection exceeds the capacity is redone by the workgroup of its
// first chunk.
//
// Measured, us per call, 8 heads.  One workgroup, against three passes of 12, 12 and 8 bits over all scores (count and mass apart): 18763 scores
// 36.5 -> 23.4, 8192 24.4 -> 14.6, 4096 19.2 -> 14.6 (the kernel alone 17.7 -> 9; two launches take the host 14).  Many, against the same passes in
// seven kernels / a list of the candidates in the workspace instead of the third kernel, which every workgroup then reads, or all scores where it
// does not hold them: 131072 scores of a wide spread 49 / 27 -> 30, within 2 percent of each other 70 / 67 -> 35, equal 82 / 34 -> 25, 342475 wide
// 89 / 49 -> 52, within 2 percent 199 / 170 -> 67; one head 342475 wide 44 / 46 -> 30, within 2 percent 66 / 161 -> 35.  The five kernels of 8 x 131072
// take 2.4 + 5.2 + 7.8 + 5.6 + 9.4 us.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "vs_common.h"
#include "vs_wave.h"

namespace {

constexpr int kSelThreads = 1024;
constexpr int kWaves = kSelThreads / 64;
constexpr int kTopShift = 19, kTopBuckets = 2048;             // first digit
constexpr int kDigit = 10, kDigitBuckets = 1 << kDigit;       // digits below
constexpr int kBatch = 8;                      // scores per lane that are requested together
constexpr int kMinSplitN = 32768;              // shorter problems stay with one workgroup (fewer launches)
typedef unsigned long long u64;

struct SelParams {
    const float* a[2];
    int32_t* idx[2];
    int32_t* cnt[2];
    int32_t* status;
    int n, mode;
    double tau[2];
    int kfix[2], nforced[2], cap[2];
};

__device__ __forceinline__ uint32_t score_key(float x, int& st) {
    if (!(x >= 0.f)) {            // NaN or negative
        st |= VS_STATUS_BAD_SCORE;
        return 0u;
    }
    const uint32_t key = x == 0.f ? 0u : __float_as_uint(x);
    if (key > 0x3f800000u) st |= VS_STATUS_SATURATED;
    return key;
}
__device__ __forceinline__ uint32_t score_key(float x) {
    int dummy = 0;
    return score_key(x, dummy);
}

// floor(min(score, 1) * 2^40) from the bits: the significand moved by the exponent
__device__ __forceinline__ u64 key_mass(uint32_t key) {
    key = min(key, 0x3f800000u);
    const uint32_t down = 127u - (key >> 23);
    return down > 63u ? 0ull : (static_cast<u64>((key & 0x7fffffu) | 0x800000u) << 17) >> down;
}

__device__ __forceinline__ uint32_t top_bucket(uint32_t key) { return min(key >> kTopShift, static_cast<uint32_t>(kTopBuckets - 1)); }

// A histogram in LDS: R buckets per lane of the scanning wavefront, from the highest bucket down; neighbouring buckets, which the
// scores crowd into, lie 65 entries apart (different banks), and the scan's reads are conflict-free.
template <int NB>
struct Hist {
    static constexpr int kPerLane = NB / 64, kWords = kPerLane * 65;
    static __device__ __forceinline__ int slot(uint32_t b) {
        const uint32_t r = NB - 1 - b;
        return static_cast<int>((r % kPerLane) * 65 + r / kPerLane);
    }
};
constexpr int kHistWords = Hist<kTopBuckets>::kWords;

template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_moved(T x) {
    if constexpr (sizeof(T) == 8) {
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false);
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(x >> 32), CTRL, ROWS, 0xf, false);
        return (static_cast<u64>(hi) << 32) | lo;
    } else {
        return __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false);
    }
}
// inclusive sum over the lanes (row shifts, then the last lane of a row and of a half handed on); all lanes active
template <typename T>
__device__ __forceinline__ T wave_scan(T x) {
    x += dpp_moved<0x111, 0xf>(x);
    x += dpp_moved<0x112, 0xf>(x);
    x += dpp_moved<0x114, 0xf>(x);
    x += dpp_moved<0x118, 0xf>(x);
    x += dpp_moved<0x142, 0xa>(x);
    x += dpp_moved<0x143, 0xc>(x);
    return x;
}
template <typename T>
__device__ __forceinline__ T lane_value(T x, int lane) {      // lane: wave-uniform
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(x), lane);
    if constexpr (sizeof(T) == 4) return static_cast<T>(lo);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(static_cast<u64>(x) >> 32), lane);
    return static_cast<T>((static_cast<u64>(hi) << 32) | lo);
}

// State of a problem's descent.
struct Descent {
    u64 target;            // weight that the elements not above the prefix still have to contribute
    uint32_t bucket;       // crossing bucket of the last digit
    uint32_t none, all;    // nothing / everything is in by rank
};

// Called by wavefront 0: the bucket in which the running weight, from the highest bucket down, reaches the target.  tau >= 0 (first
// digit of the threshold rule, whose histogram has every element): the target is ceil(tau * total).
template <int NB>
__device__ __forceinline__ void find_crossing(const u64* hist, double tau, Descent& d) {
    constexpr int R = Hist<NB>::kPerLane;
    const int lane = threadIdx.x & 63;
    u64 sum = 0;
#pragma unroll
    for (int j = 0; j < R; ++j) sum += hist[j * 65 + lane];
    const u64 incl = wave_scan(sum);
    if (tau >= 0.0) {
        const u64 total = lane_value(incl, 63);
        d.target = static_cast<u64>(ceil(tau * static_cast<double>(total)));
        if (d.target == 0) {
            d.none = 1u;
            return;
        }
        if (d.target > total) {
            // Totals above 2^53 are rounded when they become a double, so ceil(tau * total) can exceed the total itself (tau = 1, more
            // than 2^13 saturated scores): the mass is then never reached and the rule keeps every element.
            d.all = 1u;
            d.bucket = 0u;
            return;
        }
    }
    const u64 hit = __ballot(incl - sum < d.target && incl >= d.target);
    const int l = hit ? __builtin_ctzll(hit) : 63;
    const u64 base = lane_value(incl - sum, l);
    const u64 mine = lane < R ? hist[lane * 65 + l] : 0ull;
    const u64 upto = base + wave_scan(mine);
    const u64 hit2 = __ballot(lane < R && upto - mine < d.target && upto >= d.target);
    const int j = hit2 ? __builtin_ctzll(hit2) : R - 1;
    d.target -= lane_value(upto - mine, j);
    d.bucket = static_cast<uint32_t>(NB - 1 - (l * R + j));
}

// Bits of a key below its top bucket (the last bucket has everything above); key - low_end() has that many.
__device__ __forceinline__ int bits_below(uint32_t top) { return top == kTopBuckets - 1 ? 30 : kTopShift; }
__device__ __forceinline__ uint32_t low_end(uint32_t top) { return top << kTopShift; }

// The remaining `bits` bits, kDigit at a time: each(f) calls f(candidate, valid) (candidate: key, bit 31: forced) for the candidates that
// share the bits above (prefix).  Returns key - low; d.target is then the weight that the ties at it contribute.  All threads of
// the workgroup.
template <typename EACH>
__device__ __forceinline__ uint32_t descend(u64* hist, Descent* shared, Descent& d, uint32_t low, uint32_t prefix, int bits, bool by_count,
                                            EACH each) {
    const int tid = threadIdx.x;
    while (bits > 0) {
        const int shf = bits > kDigit ? bits - kDigit : 0;
        for (int b = tid; b < Hist<kDigitBuckets>::kWords; b += kSelThreads) hist[b] = 0ull;
        __syncthreads();
        each([&](uint32_t cand, bool valid) __attribute__((always_inline)) {
            const uint32_t key = cand & 0x7fffffffu, rel = key - low;
            if (valid && (rel >> bits) == prefix)
                atomicAdd(&hist[Hist<kDigitBuckets>::slot((rel >> shf) & ((1u << (bits - shf)) - 1))],
                          by_count ? 1ull : key_mass(key));
        });
        __syncthreads();
        if (tid < 64) {
            find_crossing<kDigitBuckets>(hist, -1.0, d);
            if (tid == 0) *shared = d;
        }
        __syncthreads();
        d = *shared;
        prefix = (prefix << (bits - shf)) | d.bucket;
        bits = shf;
    }
    return prefix;
}

// ties at the crossing value that are in: the fewest whose weight reaches the target (every tie has the same weight)
__device__ __forceinline__ uint32_t ties_taken(const Descent& d, uint32_t vstar, bool by_count) {
    if (by_count) return static_cast<uint32_t>(d.target);
    const u64 w = key_mass(vstar);
    return static_cast<uint32_t>((d.target + w - 1) / w);
}

// Entries of a part (a wavefront's range, a chunk) that are in whatever the ties decide, ties, forced ties; ties are taken in index
// order and the forced entries, already counted as in, are the lowest indices: the number of selected entries follows.
__device__ __forceinline__ uint32_t part_selected(uint32_t in, uint32_t eq, uint32_t eqf, uint32_t ties_before, uint32_t ties) {
    const uint32_t room = ties > ties_before + eqf ? ties - ties_before - eqf : 0u;
    return in + min(room, eq - eqf);
}

// This wavefront's scores [lo, hi) in batches of 64 * kBatch; a range of one batch is requested once and stays in registers.
struct Range {
    const float* a;
    int lo, hi, have;
    float x[kBatch];
    __device__ __forceinline__ Range(const float* scores, int lo_, int hi_) : a(scores), lo(lo_), hi(hi_), have(-1) {
        if (lo < hi) load(lo);
    }
    __device__ __forceinline__ void load(int base) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) x[j] = a[min(base + 64 * j + lane, hi - 1)];
        have = base;
    }
    // f(index, score, valid) for all lanes of the wavefront, 64 scores at a time
    template <typename F>
    __device__ __forceinline__ void each(F f) {
        each(f, [](int, int, float) __attribute__((always_inline)) { return false; });
    }
    // The same, but first same(index of the first, number, score) for a batch of equal scores, which returns whether that was all:
    // atomics of a wavefront on one LDS word are served one after the other (8 heads x 131072 equal scores 45 us per call without it).
    template <typename F, typename G>
    __device__ __forceinline__ void each(F f, G same) {
        const int lane = threadIdx.x & 63;
        for (int base = lo; base < hi; base += 64 * kBatch) {
            if (base != have) load(base);
            const uint32_t first = __builtin_amdgcn_readfirstlane(__float_as_uint(x[0]));
            bool equal = true;
#pragma unroll
            for (int j = 0; j < kBatch; ++j) equal &= __float_as_uint(x[j]) == first;
            if (__all(equal) && same(base, min(hi - base, 64 * kBatch), __uint_as_float(first))) continue;
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int i = base + 64 * j + lane;
                if (base + 64 * j < hi) f(i, x[j], i < hi);
            }
        }
    }
};

struct SelShared {
    u64 hist[kHistWords];
    Descent descent;
    uint32_t in[kWaves], eq[kWaves], eqf[kWaves];
    int status;
};

// Ascending output of one wavefront's range: pos and tie_run are those of its first entry.
template <typename RANKED>
__device__ __forceinline__ void emit(Range& r, int32_t* __restrict__ out, uint32_t pos, uint32_t tie_run, uint32_t vstar, uint32_t ties, int nforced,
                                     RANKED ranked) {
    const u64 lt_mask = (1ull << (threadIdx.x & 63)) - 1ull;
    r.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
        const uint32_t key = score_key(x);
        const bool rk = valid && ranked(i);
        const bool eq = rk && key == vstar;
        bool in = (valid && i < nforced) || (rk && key > vstar);
        const u64 eb = __ballot(eq);
        if (eq && tie_run + __popcll(eb & lt_mask) < ties) in = true;
        tie_run += __popcll(eb);
        const u64 sb = __ballot(in);
        if (in) out[pos + __popcll(sb & lt_mask)] = i;
        pos += __popcll(sb);
    });
}

// One problem by one workgroup.  STORED: the candidates go to cand (as many entries as scores), else they are looked for among the
// scores again.  overflowed: the selection is known to exceed the capacity.
template <bool STORED>
__device__ void select_problem(const SelParams& p, int head, int dir, SelShared& sh, uint32_t* cand, bool overflowed) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = p.n, nforced = min(p.nforced[dir], n), cap = p.cap[dir];
    const u64 lt_mask = (1ull << lane) - 1ull;
    const int per_wave = ((n + kWaves - 1) / kWaves + 63) & ~63;
    const int w_lo = min(wave * per_wave, n), w_hi = min(w_lo + per_wave, n);
    Range range(p.a[dir] + static_cast<size_t>(head) * n, w_lo, w_hi);
    int st = overflowed ? VS_STATUS_OVERFLOW : 0;
    if (tid == 0) sh.status = 0;
    bool by_count = p.mode != 0;
    // The second attempt keeps the forced entries and fills up with the best-ranked others: a pick by count over the rest.
    for (int attempt = overflowed ? 1 : 0; attempt < 2; ++attempt) {
        const bool skip_forced = attempt != 0;
        Descent d{};
        if (skip_forced) by_count = true;
        const bool collect = !skip_forced;                   // status bits of the scores
        if (by_count) {
            d.target = skip_forced ? static_cast<u64>(cap - nforced) : static_cast<u64>(min(p.kfix[dir], n));
            d.none = d.target == 0 ? 1u : 0u;
        }
        auto ranked = [&](int i) __attribute__((always_inline)) { return !d.none && !(skip_forced && i < nforced); };
        for (int b = tid; b < kHistWords; b += kSelThreads) sh.hist[b] = 0ull;
        __syncthreads();
        range.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
            if (!valid) return;
            int bits = 0;
            const uint32_t key = score_key(x, bits);
            if (collect) st |= bits;
            if (ranked(i)) {
                const u64 w = by_count ? 1ull : key_mass(key);
                if (w) atomicAdd(&sh.hist[Hist<kTopBuckets>::slot(top_bucket(key))], w);
            }
        });
        __syncthreads();
        if (tid < 64) {
            if (!d.none) find_crossing<kTopBuckets>(sh.hist, by_count ? -1.0 : p.tau[dir], d);
            if (tid == 0) sh.descent = d;
        }
        __syncthreads();
        d = sh.descent;
        const uint32_t top = d.bucket;
        // candidates of this wavefront, at w_lo of cand on; entries above them and forced ones are in
        uint32_t inc = 0, mine = 0;
        range.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
            const uint32_t key = score_key(x), b = top_bucket(key);
            const bool forced = valid && i < nforced, rk = valid && ranked(i);
            const bool c = rk && b == top;
            inc += __popcll(__ballot(forced || (rk && b > top)));
            const u64 cb = __ballot(c);
            if (STORED && c) cand[w_lo + mine + __popcll(cb & lt_mask)] = key | (forced ? 0x80000000u : 0u);
            mine += __popcll(cb);
        });
        auto each = [&](auto f) __attribute__((always_inline)) {
            if constexpr (STORED) {
                for (uint32_t k = 0; k < mine; k += 64) f(k + lane < mine ? cand[w_lo + k + lane] : 0u, k + lane < mine);
            } else {
                range.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
                    const uint32_t key = score_key(x);
                    f(key | (i < nforced ? 0x80000000u : 0u), valid && ranked(i) && top_bucket(key) == top);
                });
            }
        };
        uint32_t vstar = 0u, ties = 0xffffffffu;             // everything is in: crossing value 0 and every tie
        if (d.none) ties = 0u;
        else if (!d.all) {
            vstar = low_end(top) + descend(sh.hist, &sh.descent, d, low_end(top), 0u, bits_below(top), by_count, each);
            ties = ties_taken(d, vstar, by_count);
        }
        uint32_t eqc = 0, eqf = 0, above = 0;
        each([&](uint32_t c, bool valid) __attribute__((always_inline)) {
            const uint32_t key = c & 0x7fffffffu, forced = c >> 31;
            eqc += valid && key == vstar ? 1u : 0u;
            eqf += valid && key == vstar ? forced : 0u;
            above += valid && key > vstar ? 1u - forced : 0u;
        });
        // (three counts below 2^21 each: two sums over the lanes)
        const u64 sums = wave_scan((static_cast<u64>(eqc) << 32) | eqf);
        const uint32_t more = wave_scan(above);
        if (lane == 63) {
            sh.eq[wave] = static_cast<uint32_t>(sums >> 32);
            sh.eqf[wave] = static_cast<uint32_t>(sums);
            sh.in[wave] = inc + more;
        }
        __syncthreads();
        const uint32_t e = lane < kWaves ? sh.eq[lane] : 0u, ef = lane < kWaves ? sh.eqf[lane] : 0u, in = lane < kWaves ? sh.in[lane] : 0u;
        const uint32_t ties_before = wave_scan(e) - e;
        const uint32_t sel = part_selected(in, e, ef, ties_before, ties);
        const uint32_t upto = wave_scan(sel);
        const uint32_t total = lane_value(upto, 63);
        if (total > static_cast<uint32_t>(cap) && attempt == 0) {
            st |= VS_STATUS_OVERFLOW;
            continue;
        }
        emit(range, p.idx[dir] + static_cast<size_t>(head) * cap, lane_value(upto - sel, wave), lane_value(ties_before, wave), vstar, ties, nforced,
             ranked);
        if (tid == 0) p.cnt[dir][head] = static_cast<int32_t>(total);
        break;
    }
    if (st) atomicOr(&sh.status, st);
    __syncthreads();
    if (tid == 0 && p.status && sh.status) atomicOr(p.status + head, sh.status);
}

template <bool STORED>
__global__ __launch_bounds__(kSelThreads) void select_kernel(const SelParams p) {
    __shared__ SelShared sh;
    extern __shared__ uint32_t cand[];
    select_problem<STORED>(p, blockIdx.x, blockIdx.y, sh, cand, false);
}

// ---- the same selection over many workgroups ----
constexpr int kChunk = 8192;                   // scores per workgroup up to 524288, one batch of every wavefront; longer problems have longer chunks
constexpr int kMaxChunks = 64;                 // a lane per chunk adds up the positions
static_assert(kChunk == kSelThreads * kBatch, "one batch");
// digits of a key: 11, 11 and 9 bits
constexpr int kShift1 = 20, kShift2 = 9, kBuckets = 2048, kLastBuckets = 1 << kShift2;
static_assert(kHistWords == Hist<kBuckets>::kWords, "one histogram");

// Workspace of one problem.  The histograms are 64 lanes wide, otherwise as in LDS: neighbouring buckets are 512 bytes apart, and atomics
// of many workgroups on one line, which are served one after the other, are few.
struct ProblemWs {
    u64 hist[kBuckets], next[kBuckets];        // first digit; second digit in the crossing bucket of the first
};
struct ProblemState {
    Descent first, second;                     // after these digits; second.bucket: both digits
};
// What a workgroup finds in its chunk
struct ChunkWs {
    uint32_t in;                               // forced entries, and those above the crossing bucket of the first digit
    uint32_t above;                            // unforced ones in that, above the crossing bucket of the second
    uint32_t pad[62];
    uint32_t last[kLastBuckets];               // those in that by their last digit; unforced ones also count in the high half
};
constexpr int kLongestChunk = 7 * kChunk;
static_assert(kLongestChunk < 65536 && VS_MAX_SEQ <= kMaxChunks * kLongestChunk, "two counts in a word");
struct SplitParams {
    SelParams s;
    int chunks, chunk_size;                    // chunk_size: a multiple of kChunk
    ProblemWs* problem;
    ProblemState* state;
    ChunkWs* chunk;                            // [problems][chunks]
};

// This wavefront's scores of the workgroup's chunk
__device__ __forceinline__ Range chunk_range(const SplitParams& q, int wave) {
    const int n = q.s.n, per_wave = q.chunk_size / kWaves;
    const int lo = min(static_cast<int>(blockIdx.x) * q.chunk_size + wave * per_wave, n);
    return Range(q.s.a[blockIdx.z] + static_cast<size_t>(blockIdx.y) * n, lo, min(lo + per_wave, n));
}

__device__ __forceinline__ void add_histogram(const u64* hist, u64* out) {
    for (int r = threadIdx.x; r < kBuckets; r += kSelThreads) {
        const u64 w = hist[(r >> 6) * 65 + (r & 63)];         // both layouts have 64 lanes
        if (w) atomicAdd(&out[r], w);
    }
}
__device__ __forceinline__ void load_histogram(const u64* in, u64* hist) {
    for (int r = threadIdx.x; r < kBuckets; r += kSelThreads) hist[(r >> 6) * 65 + (r & 63)] = in[r];
}

__global__ __launch_bounds__(kSelThreads) void split_first_kernel(const SplitParams q) {
    __shared__ u64 hist[kHistWords];
    const SelParams& p = q.s;
    const int head = blockIdx.y, dir = blockIdx.z, tid = threadIdx.x;
    const bool by_count = p.mode != 0;
    Range range = chunk_range(q, __builtin_amdgcn_readfirstlane(tid >> 6));
    for (int b = tid; b < kHistWords; b += kSelThreads) hist[b] = 0ull;
    __syncthreads();
    int st = 0;
    range.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
        if (!valid) return;
        const uint32_t key = score_key(x, st);
        const u64 w = by_count ? 1ull : key_mass(key);
        if (w) atomicAdd(&hist[Hist<kBuckets>::slot(key >> kShift1)], w);
    }, [&](int, int num, float x) __attribute__((always_inline)) {
        const uint32_t key = score_key(x, st);
        if ((tid & 63) == 0) atomicAdd(&hist[Hist<kBuckets>::slot(key >> kShift1)], num * (by_count ? 1ull : key_mass(key)));
        return true;
    });
    if (st && p.status) atomicOr(p.status + head, st);
    __syncthreads();
    add_histogram(hist, q.problem[head * 2 + dir].hist);
}

// The crossing bucket of the first digit, and the histogram of the second digit in it.
__global__ __launch_bounds__(kSelThreads) void split_second_kernel(const SplitParams q) {
    __shared__ u64 hist[kHistWords], next[kHistWords];
    __shared__ Descent shared;
    __shared__ uint32_t part[kWaves];
    const SelParams& p = q.s;
    const int chunk = blockIdx.x, head = blockIdx.y, dir = blockIdx.z, pr = head * 2 + dir;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nforced = min(p.nforced[dir], p.n);
    const bool by_count = p.mode != 0;
    Range range = chunk_range(q, wave);
    load_histogram(q.problem[pr].hist, hist);
    for (int b = tid; b < kHistWords; b += kSelThreads) next[b] = 0ull;
    __syncthreads();
    Descent d{};
    if (by_count) {
        d.target = static_cast<u64>(min(p.kfix[dir], p.n));
        d.none = d.target == 0 ? 1u : 0u;
    }
    if (tid < 64) {
        if (!d.none) find_crossing<kBuckets>(hist, by_count ? -1.0 : p.tau[dir], d);
        if (tid == 0) {
            shared = d;
            if (chunk == 0) q.state[pr].first = d;
        }
    }
    __syncthreads();
    d = shared;
    uint32_t inc = 0;
    range.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
        const uint32_t key = score_key(x), b = key >> kShift1;
        inc += __popcll(__ballot(valid && (i < nforced || (!d.none && b > d.bucket))));
        if (valid && !d.none && b == d.bucket) {
            const u64 w = by_count ? 1ull : key_mass(key);
            if (w) atomicAdd(&next[Hist<kBuckets>::slot((key >> kShift2) & (kBuckets - 1))], w);
        }
    }, [&](int base, int num, float x) __attribute__((always_inline)) {
        const uint32_t key = score_key(x), b = key >> kShift1;
        inc += !d.none && b > d.bucket ? num : min(max(nforced - base, 0), num);
        if (lane == 0 && !d.none && b == d.bucket)
            atomicAdd(&next[Hist<kBuckets>::slot((key >> kShift2) & (kBuckets - 1))], num * (by_count ? 1ull : key_mass(key)));
        return true;
    });
    if (lane == 0) part[wave] = inc;
    __syncthreads();
    if (tid < 64) {
        inc = wave_scan(lane < kWaves ? part[lane] : 0u);
        if (lane == 63) q.chunk[static_cast<size_t>(pr) * q.chunks + chunk].in = inc;
    }
    add_histogram(next, q.problem[pr].next);
}

// The crossing bucket of the second digit, and this chunk's entries of it by their last digit.
__global__ __launch_bounds__(kSelThreads) void split_last_kernel(const SplitParams q) {
    __shared__ u64 hist[kHistWords];
    __shared__ uint32_t last[kLastBuckets], part[kWaves];
    __shared__ Descent shared;
    const SelParams& p = q.s;
    const int chunk = blockIdx.x, head = blockIdx.y, dir = blockIdx.z, pr = head * 2 + dir;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nforced = min(p.nforced[dir], p.n);
    Range range = chunk_range(q, wave);
    load_histogram(q.problem[pr].next, hist);
    Descent d = q.state[pr].first;
    if (d.none || d.all) return;
    if (tid < kLastBuckets) last[tid] = 0u;
    __syncthreads();
    const uint32_t first = d.bucket;
    if (tid < 64) {
        find_crossing<kBuckets>(hist, -1.0, d);
        d.bucket |= first << (kShift1 - kShift2);
        if (tid == 0) {
            shared = d;
            if (chunk == 0) q.state[pr].second = d;
        }
    }
    __syncthreads();
    const uint32_t prefix = shared.bucket;
    uint32_t above = 0;
    range.each([&](int i, float x, bool valid) __attribute__((always_inline)) {
        const uint32_t key = score_key(x), b = key >> kShift2;
        const bool forced = i < nforced;
        above += __popcll(__ballot(valid && !forced && b > prefix && (key >> kShift1) == first));
        if (valid && b == prefix) atomicAdd(&last[key & (kLastBuckets - 1)], forced ? 1u : 0x10001u);
    }, [&](int base, int num, float x) __attribute__((always_inline)) {
        const uint32_t key = score_key(x), b = key >> kShift2, unforced = num - min(max(nforced - base, 0), num);
        if (b > prefix && (key >> kShift1) == first) above += unforced;
        if (lane == 0 && b == prefix) atomicAdd(&last[key & (kLastBuckets - 1)], (unforced << 16) + num);
        return true;
    });
    if (lane == 0) part[wave] = above;
    __syncthreads();
    ChunkWs& out = q.chunk[static_cast<size_t>(pr) * q.chunks + chunk];
    if (tid < kLastBuckets) out.last[tid] = last[tid];
    if (tid < 64) {
        above = wave_scan(lane < kWaves ? part[lane] : 0u);
        if (lane == 63) out.above = above;
    }
}

// The crossing value and the ordered emission of a chunk.
__global__ __launch_bounds__(kSelThreads) void split_emit_kernel(const SplitParams q) {
    __shared__ SelShared sh;
    __shared__ uint32_t c_in[kMaxChunks], c_eq[kMaxChunks], c_ef[kMaxChunks];
    const SelParams& p = q.s;
    const int chunk = blockIdx.x, head = blockIdx.y, dir = blockIdx.z, pr = head * 2 + dir;
    const int tid = threadIdx.x, lane = tid & 63, n = p.n;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nforced = min(p.nforced[dir], n);
    const bool by_count = p.mode != 0;
    const ChunkWs* const info = q.chunk + static_cast<size_t>(pr) * q.chunks;
    Range range = chunk_range(q, wave);
    // a wavefront adds up every sixteenth chunk; what it needs of the first is requested here (the words of a chunk without a last digit
    // hold anything and are not looked at)
    constexpr int kEntries = kLastBuckets / 64;
    uint32_t num[kEntries], in_above = 0;
    auto request = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kEntries; ++j) num[j] = info[c].last[64 * j + lane];
        in_above = info[c].in + info[c].above;
    };
    request(min(wave, q.chunks - 1));
    const Descent second = q.state[pr].second;
    Descent d = q.state[pr].first;
    uint32_t vstar = 0u, ties = 0xffffffffu;                 // everything is in: crossing value 0 and every tie
    if (d.none || d.all) {
        if (d.none) ties = 0u;
        if (tid < q.chunks) {
            c_in[tid] = d.none ? info[tid].in : static_cast<uint32_t>(min(q.chunk_size, n - tid * q.chunk_size));
            c_eq[tid] = c_ef[tid] = 0u;
        }
    } else {
        d = second;
        const uint32_t low = d.bucket << kShift2;
        // All entries of a last bucket have the same weight, so that counts are enough.
        for (int b = tid; b < Hist<kLastBuckets>::kWords; b += kSelThreads) sh.hist[b] = 0ull;
        __syncthreads();
        for (int c = wave; c < q.chunks; c += kWaves) {
            if (c != wave) request(c);
#pragma unroll
            for (int j = 0; j < kEntries; ++j) {
                const uint32_t b = 64 * j + lane, all = num[j] & 0xffffu;
                if (all) atomicAdd(&sh.hist[Hist<kLastBuckets>::slot(b)], by_count ? all : all * key_mass(low + b));
            }
        }
        __syncthreads();
        if (tid < 64) {
            find_crossing<kLastBuckets>(sh.hist, -1.0, d);
            if (tid == 0) sh.descent = d;
        }
        __syncthreads();
        d = sh.descent;
        vstar = low + d.bucket;
        ties = ties_taken(d, vstar, by_count);
        for (int c = wave; c < q.chunks; c += kWaves) {
            if (q.chunks > kWaves) request(c);
            uint32_t more = 0, eq = 0;
#pragma unroll
            for (int j = 0; j < kEntries; ++j) {
                const uint32_t b = 64 * j + lane;
                more += b > d.bucket ? num[j] >> 16 : 0u;
                eq += b == d.bucket ? num[j] : 0u;
            }
            more = wave_scan(more);
            eq = wave_scan(eq);
            if (lane == 63) {
                c_in[c] = in_above + more;
                c_eq[c] = eq & 0xffffu;
                c_ef[c] = (eq & 0xffffu) - (eq >> 16);
            }
        }
    }
    // this wavefront's range of this chunk
    uint32_t w_eq = 0, w_ef = 0, w_in = 0;
    range.each([&](int i, float s, bool valid) __attribute__((always_inline)) {
        const uint32_t key = score_key(s);
        const bool forced = valid && i < nforced, rk = valid && !d.none;
        const bool eq = rk && key == vstar;
        w_eq += __popcll(__ballot(eq));
        w_ef += __popcll(__ballot(eq && forced));
        w_in += __popcll(__ballot(forced || (rk && key > vstar)));
    });
    if (lane == 0) {
        sh.eq[wave] = w_eq;
        sh.eqf[wave] = w_ef;
        sh.in[wave] = w_in;
    }
    __syncthreads();
    // positions: first of the chunks, then of the wavefronts inside this one
    const bool is = lane < q.chunks;
    uint32_t e = is ? c_eq[lane] : 0u;
    uint32_t before = wave_scan(e) - e;
    uint32_t sel = part_selected(is ? c_in[lane] : 0u, e, is ? c_ef[lane] : 0u, before, ties);
    uint32_t pos = wave_scan(sel);
    const uint32_t total = lane_value(pos, 63);
    if (total > static_cast<uint32_t>(p.cap[dir])) {         // redone by one workgroup
        if (chunk == 0) select_problem<false>(p, head, dir, sh, nullptr, true);
        return;
    }
    if (chunk == 0 && tid == 0) p.cnt[dir][head] = static_cast<int32_t>(total);
    const uint32_t chunk_before = lane_value(before, chunk), chunk_pos = lane_value(pos - sel, chunk);
    const bool iw = lane < kWaves;
    e = iw ? sh.eq[lane] : 0u;
    before = chunk_before + wave_scan(e) - e;
    sel = part_selected(iw ? sh.in[lane] : 0u, e, iw ? sh.eqf[lane] : 0u, before, ties);
    pos = chunk_pos + wave_scan(sel) - sel;
    emit(range, p.idx[dir] + static_cast<size_t>(head) * p.cap[dir], lane_value(pos, wave), lane_value(before, wave), vstar, ties, nforced,
         [&](int) __attribute__((always_inline)) { return !d.none; });
}

// Histograms of the problems, status words
__global__ __launch_bounds__(kSelThreads) void clear_kernel(ProblemWs* problem, int32_t* status) {
    uint4* const w = reinterpret_cast<uint4*>(problem + blockIdx.x);
    for (int i = threadIdx.x; i < static_cast<int>(sizeof(ProblemWs) / 16); i += kSelThreads) w[i] = make_uint4(0u, 0u, 0u, 0u);
    if (status && threadIdx.x == 0 && (blockIdx.x & 1) == 0) status[blockIdx.x >> 1] = 0;
}

struct SplitLayout {
    size_t state, chunk, total, size;      // total: what a call uses; size: what the query says
    int chunks, chunk_size;
};

SplitLayout split_layout(int heads, int64_t n) {
    SplitLayout w{};
    const size_t pr = static_cast<size_t>(heads) * 2;
    // Up to 131072 scores chunks of 8192.  Beyond, the length with the least work for the busiest of 256 compute units (a workgroup costs about
    // as much as 8192 scores more), of equal ones the longest: every workgroup looks at what all chunks of its problem have found.  us per call: 8 heads x 2^20 in 19 chunks (304 workgroups) 141, 32
    // (512) 97, 64 110; 8 x 342475 in 21 chunks (336) 59, 14 (224) 52; 32 x 342475 in 42 chunks 167, 11 (704) 129.
    int64_t least = INT64_MAX;
    for (int size = kChunk; size <= kLongestChunk; size += kChunk) {
        const int64_t chunks = (n + size - 1) / size, work = (static_cast<int64_t>(pr) * chunks + 255) / 256 * (size + kChunk);
        if (chunks > kMaxChunks || work > least) continue;
        least = work;
        w.chunk_size = size;
        w.chunks = static_cast<int>(chunks);
        if (n <= 131072) break;
    }
    w.state = pr * sizeof(ProblemWs);
    w.chunk = vs::round_up(w.state + pr * sizeof(ProblemState), 256);
    w.total = w.chunk + pr * w.chunks * sizeof(ChunkWs);
    // The query's answer grows with n (a workspace for n does for shorter problems) and is never less than when a problem had three
    // histograms of 4096 entries.
    const int64_t short_chunks = (n + kChunk - 1) / kChunk;
    const size_t former = vs::round_up(pr * (3 * 4096 * 12 + 4), 256) + vs::round_up(pr * 192, 256) + vs::round_up(pr * short_chunks * 12, 256);
    w.size = std::max(former, w.chunk + pr * std::min<int64_t>(kMaxChunks, short_chunks) * sizeof(ChunkWs));
    return w;
}

__global__ void zero_status_kernel(int32_t* status, int heads) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < heads) status[i] = 0;
}

}  // namespace

extern "C" {

size_t vs_select_budget_workspace(int heads, int64_t n) {
    if (heads <= 0 || n < kMinSplitN || n > VS_MAX_SEQ) return 0;   // one workgroup per problem: everything lives in LDS
    return split_layout(heads, n).size;
}

int vs_select_budget(const float* a_v, const float* a_s, int heads, int64_t n, const vs_budget_t* b, int32_t* idx_v,
                     int32_t* cnt_v, int32_t* idx_s, int32_t* cnt_s, int32_t* status, void* ws, size_t ws_bytes,
                     void* stream) {
    if (!a_v || !a_s || !b || !idx_v || !cnt_v || !idx_s || !cnt_s) return VS_ERR_INVALID_ARG;
    if (heads <= 0 || n <= 0) return VS_ERR_INVALID_ARG;
    if (n > VS_MAX_SEQ || heads > 65535) return VS_ERR_UNSUPPORTED;
    if (b->mode != 0 && b->mode != 1) return VS_ERR_INVALID_ARG;
    if (b->mode == 0 && !(b->tau_v >= 0.0 && b->tau_v <= 1.0 && b->tau_s >= 0.0 && b->tau_s <= 1.0)) return VS_ERR_INVALID_ARG;
    if (b->mode == 1 && (b->k_v < 0 || b->k_s < 0)) return VS_ERR_INVALID_ARG;
    if (b->n_sink < 0) return VS_ERR_INVALID_ARG;
    if (b->cap_v <= 0 || b->cap_s <= 0) return VS_ERR_CAPACITY;
    const int64_t forced_v = b->n_sink < n ? b->n_sink : n;
    const int64_t local = b->n_local < 1 ? 1 : b->n_local;
    const int64_t forced_s = local < n ? local : n;
    if (forced_v > b->cap_v || forced_s > b->cap_s) return VS_ERR_CAPACITY;

    SelParams p{};
    p.a[0] = a_v;
    p.a[1] = a_s;
    p.idx[0] = idx_v;
    p.idx[1] = idx_s;
    p.cnt[0] = cnt_v;
    p.cnt[1] = cnt_s;
    p.status = status;
    p.n = static_cast<int>(n);
    p.mode = b->mode;
    p.tau[0] = b->tau_v;
    p.tau[1] = b->tau_s;
    p.kfix[0] = b->k_v;
    p.kfix[1] = b->k_s;
    p.nforced[0] = static_cast<int>(forced_v);
    p.nforced[1] = static_cast<int>(forced_s);
    p.cap[0] = b->cap_v;
    p.cap[1] = b->cap_s;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (ws && n >= kMinSplitN) {
        const SplitLayout w = split_layout(heads, n);
        if (ws_bytes < w.total) return VS_ERR_WORKSPACE;
        if (!vs::aligned16(ws)) return VS_ERR_INVALID_ARG;
        unsigned char* base = static_cast<unsigned char*>(ws);
        SplitParams q{};
        q.s = p;
        q.chunks = w.chunks;
        q.chunk_size = w.chunk_size;
        q.problem = reinterpret_cast<ProblemWs*>(base);
        q.state = reinterpret_cast<ProblemState*>(base + w.state);
        q.chunk = reinterpret_cast<ChunkWs*>(base + w.chunk);
        hipLaunchKernelGGL(clear_kernel, dim3(2 * heads), dim3(kSelThreads), 0, st, q.problem, status);
        VS_LAUNCH_CHECK();
        const dim3 grid(w.chunks, heads, 2);
        for (void (*kernel)(SplitParams) : {&split_first_kernel, &split_second_kernel, &split_last_kernel, &split_emit_kernel}) {
            hipLaunchKernelGGL(kernel, grid, dim3(kSelThreads), 0, st, q);
            VS_LAUNCH_CHECK();
        }
        return VS_OK;
    }
    if (status) {
        hipLaunchKernelGGL(zero_status_kernel, dim3((heads + 255) / 256), dim3(256), 0, st, status, heads);
        VS_LAUNCH_CHECK();
    }
    if (n < kMinSplitN) {
        static vs::PerDeviceOnce once;
        const int rc = once.run(nullptr, [](int) -> int {
            VS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, kMinSplitN * 4));
            return VS_OK;
        });
        if (rc != VS_OK) return rc;
        hipLaunchKernelGGL(select_kernel<true>, dim3(heads, 2), dim3(kSelThreads), static_cast<size_t>(n) * 4, st, p);
    } else {
        hipLaunchKernelGGL(select_kernel<false>, dim3(heads, 2), dim3(kSelThreads), 0, st, p);
    }
    VS_LAUNCH_CHECK();
    return VS_OK;
}

}  // extern "C"
