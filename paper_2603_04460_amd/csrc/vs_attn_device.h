// Device code shared by the attention kernels of libvsprefill (sparse vertical-slash, dense causal, few row blocks) and, for the
// tile layout, the aggregation sweeps: MFMA fragment types, the LDS tile layout that they stage K / V with, the launch
// parameters and the mask / staging primitives.
#pragma once
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include "vs_common.h"
#include "vs_wave.h"

namespace vs {

struct AttnParams {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    uint16_t* o;
    float* lse;
    int q_heads, kv_heads, group, hc, n, tiles, index_per_q;   // n: keys per head
    int kv_rows;                    // vs_dense_kernel: rows of k and v per head (n: those up to the last position)
    int nq, pos0;                   // query rows per head; row r is position pos0 + r (pos0 + nq <= n)
    int gran;                       // slash granularity: 1 (element-exact) or 32 (per 32-row block)
    float scale, c;                 // c = scale * log2(e)
    const int32_t* idx_v;
    const int32_t* cnt_v;
    int cap_v;
    // prepared once per call from the index lists (one set per index head):
    const uint32_t* vbit;           // bit j set iff column j selected
    int vw;                         // words per head of vbit
    const int32_t* dlist;           // block diagonals, ascending: delta is listed iff a selected offset crosses key block
                                    // (first row block of the tile - delta) for some 32-row block of a query tile
    const unsigned long long* wlist;  // per listed diagonal and 32-row block r < 4: selected offsets 32 (delta + r) - 31 ..
                                    // 32 (delta + r) + 31 at bits 0..62
    int dcap;                       // entries per head of dlist (wlist: 4 dcap)
    const int32_t* ndiag;           // per head and 32-row block q: number of listed diagonals <= q
    const int32_t* ncol32;          // per head and 32-row block q: number of listed columns <= 32 q + 31
    int nq32;                       // entries per head of ndiag and ncol32
    const int32_t* vfirst;          // per head: position of the first non-negative entry of the column list
    unsigned long long* tile_counter;   // statistics: stat_slots groups of three counters, kStatStride apart
    int stat_slots;
    unsigned int* work_counter;     // persistent launch: next unit of every KV head's queue (zero at launch)
    int work_stride;                // counters of consecutive KV heads are this many words apart
    int work_total;                 // units of work (query tiles x KV heads x head chunks)
};

// Statistics of a sparse call (executed tiles, tiles staged by gathers and as blocks): a workgroup adds its three sums once, to
// slot blockIdx % stat_slots.  Atomics on one cache line are served one after the other, ~12 ns each, and hold up whatever else
// goes to that memory channel: with one atomic per wavefront and counter on a single line the 3072 of a small call took longer
// than the call (32 / 8 heads, n = 4096: work done after 35 us, kernel 66 us, now 48; the whole pipeline 113 -> 88 us).
constexpr int kStatStride = 16;                 // 128 bytes
constexpr int kMaxStatSlots = 64;               // 8 workgroups per slot of a full launch

// Attention for launches with few row blocks (vs_short.hip): `rows` row blocks per workgroup, 1, 2 or (sparse) 4, of p.hc =
// short_heads() query heads; the lists of a sparse call are prepared for rows / p.hc sub-blocks.
int launch_short_dense(AttnParams& p, int rows, hipStream_t stream);
int launch_short_sparse(AttnParams& p, int rows, hipStream_t stream);
inline int short_heads(int hc, int rows) { return hc < rows ? hc : rows; }
// Up to 256 row blocks, one for every compute unit, a workgroup has one row block and its eight wavefronts split the keys; beyond,
// two row blocks and four wavefronts each.  Two row blocks / one, us: dense, 1 x 8192 (256 row blocks) 74 / 45, 8 / 2 x 1024 (256)
// 15.4 / 11.6, 8 / 2 heads, 1000 rows of 65536 keys (256) 559 / 360, 64 rows, 32 / 8 heads, of 32768 (64) 280 / 151; sparse, 1 x 8192,
// 512 + 512 (256) 27.6 / 20.9, 4096 rows of 131072, 1024 + 1024 (128) 48 / 33, 1 x 1000 17.9 / 17.4.  Beyond, the second round of workgroups costs more
// than the split saves: dense 8 / 2 x 4096 (1024) 52 / 64, 32 / 8 x 500 (512) 11.6 / 13.5, 32 / 8, 500 rows of 32768 (512) 317 / 367;
// sparse 32 x 500, 62 + 62 (512) 23 / 30, 1 x 32768, 64 + 128 (1024) 38 / 51; long lists still gain (1 x 16384, 1024 + 2048 (512) 135 / 85,
// 512 + 512 33 / 35; dense 1 x 16384 142 / 104).
constexpr int kLoneBlocks = 256;
inline bool short_lone(int q_heads, int64_t nq) { return static_cast<int64_t>(q_heads) * ((nq + 31) / 32) <= kLoneBlocks; }
// Dense calls of up to 512 row blocks as well, where the second round costs nothing: a workgroup of it starts when one of the first round
// ends (longest first), and two from the middle of the order, each as long as row block 256, end before the longest does.  That is so for whole
// sequences; with a long context before the chunk all row blocks are about as long.  From 36 tiles on; the start of a workgroup costs as much as that many.
// Two row blocks (in a wavefront from 2048 keys on, else in a workgroup) / one, us: 8 / 2 x 1300 17.4 / 15.8, x 1700 21.1 / 18.8, 4 / 2 x 3000
// 25.1 / 22.0, 4 x 2800 23.1 / 19.5, 2 / 1 x 6000 39.3 / 32.9, 2 x 8000 53.6 / 52.3, 1 x 9000 53.2 / 45.4, 12000 69 / 63, 16001 97 / 98; not:
// 64 x 200 10.3 / 10.7, 16 x 800 12.7 / 14.3, 1200 rows of 8192, 8 / 2 heads 55 / 80, 9000 rows of 20000, one head 110 / 135, 8 / 2 x 2100 (528 row
// blocks) 21.6 / 25.1.
constexpr int kLoneTiles = 36;
inline bool dense_lone(int q_heads, int64_t nq, int64_t pos0) {
    if (short_lone(q_heads, nq)) return true;
    const int64_t last = (pos0 + nq + 31) / 32;
    return static_cast<int64_t>(q_heads) * ((nq + 31) / 32) <= 2 * kLoneBlocks && last >= kLoneTiles && 2 * (last - kLoneBlocks / q_heads) < last;
}

}  // namespace vs

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4t __attribute__((__vector_size__(4 * sizeof(__bf16))));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 128;
// A tile is staged with loads that write LDS directly: one wavefront instruction deposits its 64 16-byte pieces
// back to back, which makes 4 rows of 256 B a contiguous 1 KB group.  Groups are 64 B apart and the pieces are rotated
// inside a group so that fragment reads spread over all banks:
//   K (16-byte reads, 16 rows at one chunk c): chunk c of row r sits at 64 (c / 4) + 16 ((c + r) % 4) of its row
//   V (transposing reads, 4 rows x 64 B):      byte x of row r sits at 64 ((x / 64 + r) % 4) + x % 64 of its row
constexpr int kGroupBytes = 4 * 256 + 64;      // four rows and the gap to the next group
constexpr int kTileBytes = 8 * kGroupBytes;    // one 32-key tile of K or V
constexpr int kSlotBytes = 2 * kTileBytes;     // one LDS slot: a K tile, then the V tile of the same keys
constexpr int kSlots = 6;                      // ring of three stages of two tiles
constexpr uint64_t kAll63 = 0x7fffffffffffffffull;
constexpr float kRescaleThreshold = 8.0f;      // log2 units: stale maxima up to 2^8 are tolerated

using vs::AttnParams;

__device__ __forceinline__ float half_swap_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Keep-bits of one lane of a 32x32 S^T tile.  Lane (q, h) holds, in accumulator element E = 4a + c, key kj = 8a + 4h + c
// of query q; the result has that element's keep-bit at position 27 - 8a - c.
// w: selected offsets dlt-31 .. dlt+31 at bits 0..62 (key kj of row q is offset bit 31 + q - kj); cz: the causal ones
// among them; fw: keys kept for every causal row of the block; xw: keys dropped for every row.
// sh = q + 4 - 4h and ysh = 4 - 4h are per-lane constants.
__device__ __forceinline__ uint32_t lane_keep_bits(uint64_t w, uint64_t cz, uint32_t fw, uint32_t xw, int sh, int ysh) {
    const uint32_t x = static_cast<uint32_t>(w >> sh), cx = static_cast<uint32_t>(cz >> sh);
    const uint32_t yf = __builtin_bitreverse32(fw) >> ysh;  // bit 27 - 8a - c = key 8a + 4h + c
    const uint32_t yx = __builtin_bitreverse32(xw) >> ysh;
    return (x | (yf & cx)) & ~yx;
}

// Four elements (one group a) at a time: the keep-bits spread over a word each (written out: from the C form the compiler
// makes and + compare + select), then a bitwise select that stays visible to the compiler, which must space it from the
// matrix instruction that produced acc.
template <int A>
__device__ __forceinline__ void mask_elements(f32x16& acc, uint32_t keep, uint32_t dead_bits) {
    uint32_t m0, m1, m2, m3;
    asm("v_bfe_i32 %0, %4, %5, 1\n\tv_bfe_i32 %1, %4, %6, 1\n\tv_bfe_i32 %2, %4, %7, 1\n\tv_bfe_i32 %3, %4, %8, 1"
        : "=&v"(m0), "=&v"(m1), "=&v"(m2), "=&v"(m3)
        : "v"(keep), "n"(27 - 8 * A), "n"(26 - 8 * A), "n"(25 - 8 * A), "n"(24 - 8 * A));
    acc[4 * A] = __uint_as_float((m0 & __float_as_uint(acc[4 * A])) | (~m0 & dead_bits));
    acc[4 * A + 1] = __uint_as_float((m1 & __float_as_uint(acc[4 * A + 1])) | (~m1 & dead_bits));
    acc[4 * A + 2] = __uint_as_float((m2 & __float_as_uint(acc[4 * A + 2])) | (~m2 & dead_bits));
    acc[4 * A + 3] = __uint_as_float((m3 & __float_as_uint(acc[4 * A + 3])) | (~m3 & dead_bits));
    if constexpr (A + 1 < 4) mask_elements<A + 1>(acc, keep, dead_bits);
}

// Tile record of a listed key block b for one 32-row sub-block whose first position is sub_i0; w: the offset window prepared
// with the diagonal list; xw: the block's column word; n_pos: positions that exist.
//   x, y: 64-bit window wz; lane (q, h) keeps key kj iff bit 31 + q - kj of wz is set and bit kj of kw (word z) is:
//         element-exact mode: wz = selected offsets dlt-31 .. dlt+31, kw = columns not listed
//         tile-granular mode: wz = causal offsets, kw = keys that some row of the block reaches through a selected
//         offset, listed columns taken out
//   w: bit 0 live, bit 1 a mask is needed, bits 2..: the key block (so that one word per tile tells a step all it
//      needs for the staging loads and the tests; the rest is read only where a mask is applied)
__device__ __forceinline__ uint4 tile_record(int gran, int n_pos, int sub_i0, int b, uint64_t w, uint32_t xw) {
    const int dlt = sub_i0 - 32 * b;                         // offset of (row 0, key 0) of the 32x32 tile
    uint64_t wz = w;
    uint32_t kw = ~xw;
    bool live = w != 0ull, need = w != kAll63 || xw != 0u;
    if (gran == 32) {
        // Tile-granular slash: key kj is kept for every causal row of this 32-row block if ANY of its rows reaches it
        // through a selected offset, i.e. if the window has a bit in [31 - kj, 62 - kj].
        // x bit s = OR of window bits s .. s+len-1, len = rows of this block that exist (32 except at the end of
        // the sequence): doubling up to the largest power of two pw <= len, then two overlapping windows
        const int len = max(1, min(32, n_pos - sub_i0));
        uint64_t x = w;
        int pw = 1;
        while (2 * pw <= len) {
            x |= x >> pw;
            pw *= 2;
        }
        x |= x >> (len - pw);
        wz = dlt >= 31 ? kAll63 : (dlt < -31 ? 0ull : ((kAll63 << (31 - dlt)) & kAll63));   // offsets >= 0
        kw = __builtin_bitreverse32(static_cast<uint32_t>(x)) & ~xw;
        live = kw != 0u && wz != 0ull;
        need = !(kw == 0xffffffffu && wz == kAll63);
    }
    if (dlt < -31 || sub_i0 >= n_pos) live = false;          // every key lies after every row / padding rows
    return make_uint4(static_cast<uint32_t>(wz), static_cast<uint32_t>(wz >> 32), kw,
                      (live ? 1u : 0u) | (need ? 2u : 0u) | (static_cast<uint32_t>(b) << 2));
}

__device__ __forceinline__ void add_statistics(const vs::AttnParams& p, unsigned int tiles, unsigned int gather, unsigned int block) {
    unsigned long long* const c = p.tile_counter + (blockIdx.x % p.stat_slots) * vs::kStatStride;
    if (tiles) atomicAdd(c, static_cast<unsigned long long>(tiles));
    if (gather) atomicAdd(c + 1, static_cast<unsigned long long>(gather));
    if (block) atomicAdd(c + 2, static_cast<unsigned long long>(block));
}

// lds_load16 with a wave-uniform base pointer and a 32-bit per-lane byte offset: no address arithmetic per lane
__device__ __forceinline__ void lds_load16s(uint32_t voff, const void* sbase, const void* lds_base) {
    const uint32_t base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (const __attribute__((address_space(3))) void*)lds_base));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(base), "v"(voff), "s"(sbase) : "memory", "m0");
}

// The same for four rows further along a tile: the instruction's own offset moves both addresses
template <int BYTES>
__device__ __forceinline__ void lds_load16o(uint32_t voff, const void* sbase, const void* lds_base) {
    const uint32_t base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
        (const __attribute__((address_space(3))) void*)lds_base)) - BYTES;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3" : : "s"(base), "v"(voff), "s"(sbase), "n"(BYTES) : "memory", "m0");
}

// A wavefront loads the 32 rows of a tile of K or V that stand one behind the other, rows: the first of them; voff: per lane, the row
// (lane / 16) and the 16-byte chunk of the piece: no address arithmetic per load
__device__ __forceinline__ void lds_load_tile(uint32_t voff, const uint16_t* rows, unsigned char* dst) {
    lds_load16o<0>(voff, rows, dst);
    lds_load16o<1024>(voff, rows, dst + kGroupBytes);
    lds_load16o<2048>(voff, rows, dst + 2 * kGroupBytes);
    lds_load16o<3072>(voff, rows, dst + 3 * kGroupBytes);
    rows += 16 * kD;
    dst += 4 * kGroupBytes;
    lds_load16o<0>(voff, rows, dst);
    lds_load16o<1024>(voff, rows, dst + kGroupBytes);
    lds_load16o<2048>(voff, rows, dst + 2 * kGroupBytes);
    lds_load16o<3072>(voff, rows, dst + 3 * kGroupBytes);
}

// ---- stages without a row maximum ----
// Most stages of a long row block take the maximum as it stands after its first stages instead of looking for a new one: any
// value serves as long as nothing overflows or vanishes, and the precision of P, O and the sum is relative.  The sum of a lane's
// weights in the stage says whether that held: no weight is above 2^kRescaleThreshold if the sum is not.  If it is (not true for NaN, where no
// maximum helps) the stage looks for its maximum after all, the scores being at hand still, and if a row has grown by more than the threshold
// it moves the maximum and weighs its scores anew, before anything has been added to O or to the sum.  So the maximum moves where it
// would with a search in every stage, and a key whose score leaves all before it behind has a weight of exactly one.
constexpr float kGrownSum = 256.f;             // 2^kRescaleThreshold
#define VS_MAY_HAVE_GROWN(lane_sum) __builtin_expect(__ballot((lane_sum) > kGrownSum) != 0ull, 0)   // (a function loses the expectation)

// ---- row blocks whose keys are split: the partial results meet in LDS (every tile buffer is idle by then) ----
// Eight partials: O in 64 registers x 64 lanes each, then (maximum, sum) per partial and lane.
constexpr size_t kPartialStat = 8 * 64 * 64 * 4;
constexpr size_t kPartialBytes = kPartialStat + 8 * 64 * 8;

__device__ __forceinline__ void deposit_partial(unsigned char* smem, int which, const f32x16 (&oacc)[4], float m_run, float l_run) {
    const int lane = threadIdx.x & 63;
    float* const part = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) part[(which * 64 + 16 * db + e) * 64 + lane] = oacc[db][e];
    reinterpret_cast<float2*>(smem + kPartialStat)[which * 64 + lane] = make_float2(m_run, half_swap_sum(l_run));
}

// After a barrier: of a row block's SPLITS partials (first, first + stride, ..) this wavefront finishes share `split`, 128 / SPLITS channels.
template <int SPLITS>
__device__ __forceinline__ void finish_partials(const AttnParams& p, const unsigned char* smem, int first, int stride, int split, int head,
                                                int first_row) {
    const int lane = threadIdx.x & 63, qi = lane & 31, hh = lane >> 5;
    const float* const part = reinterpret_cast<const float*>(smem);
    const float2* const stat = reinterpret_cast<const float2*>(smem + kPartialStat);
    float m_tot = -INFINITY, l_tot = 0.f, f[SPLITS];
#pragma unroll
    for (int s = 0; s < SPLITS; ++s) m_tot = fmaxf(m_tot, stat[(stride * s + first) * 64 + lane].x);
#pragma unroll
    for (int s = 0; s < SPLITS; ++s) {
        const float2 x = stat[(stride * s + first) * 64 + lane];
        f[s] = x.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((x.x - m_tot) * p.c);
        l_tot = fmaf(x.y, f[s], l_tot);
    }
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    const int row = first_row + qi;
    if (row >= p.pos0 + p.nq) return;
    constexpr int kRegs = 64 / SPLITS;                       // accumulator registers that a wavefront finishes: four are 8 bytes of a row
    const int reg0 = kRegs * split;
    uint16_t* const dst = p.o + (static_cast<size_t>(head) * p.nq + (row - p.pos0)) * kD + 2 * reg0 + 4 * hh;
#pragma unroll
    for (int a = 0; a < kRegs / 4; ++a) {
        float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < SPLITS; ++s)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[c] = fmaf(part[((stride * s + first) * 64 + reg0 + 4 * a + c) * 64 + lane], f[s], x[c]);
        const f32x2 x01 = {x[0] * inv, x[1] * inv}, x23 = {x[2] * inv, x[3] * inv};
        uint2 out;
        out.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(x01, bf16x2));
        out.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(x23, bf16x2));
        *reinterpret_cast<uint2*>(dst + 8 * a) = out;
    }
    if (p.lse && split == 0 && hh == 0)
        p.lse[static_cast<size_t>(head) * p.nq + (row - p.pos0)] = l_tot > 0.f ? m_tot * p.scale + __logf(l_tot) : -INFINITY;
}

// What pads a round of the gather list (INT_MAX in LDS, masked) loads: the round's last column, a row that its tile has anyway (a weight of
// zero times a V that is not finite is NaN).  The clamp keeps undefined lists inside the buffers.
__device__ __forceinline__ int last_column(const int32_t* __restrict__ iv, int count, int n_pos) {
    return count > 0 ? max(0, min(__builtin_amdgcn_readfirstlane(iv[count - 1]), n_pos - 1)) : 0;
}

// chunk: nq query rows at positions pos0 .. pos0 + nq - 1 against n keys
int check_chunk(int64_t nq, int64_t n, int64_t pos0) {
    if (nq <= 0 || pos0 < 0 || pos0 + nq > n) return VS_ERR_INVALID_ARG;
    return VS_OK;
}

int check_qkv(const void* q, const void* k, const void* v, int q_heads, int kv_heads, int64_t n, float scale, void* o) {
    if (!q || !k || !v || !o) return VS_ERR_INVALID_ARG;
    if (!vs::aligned16(q) || !vs::aligned16(k) || !vs::aligned16(v) || !vs::aligned16(o)) return VS_ERR_INVALID_ARG;
    if (q_heads <= 0 || kv_heads <= 0 || n <= 0) return VS_ERR_INVALID_ARG;
    if (!(scale > 0.f) || !isfinite(scale)) return VS_ERR_INVALID_ARG;
    if (q_heads % kv_heads != 0) return VS_ERR_UNSUPPORTED;
    if (n > VS_MAX_SEQ) return VS_ERR_UNSUPPORTED;
    return VS_OK;
}

int heads_per_workgroup(int group, bool index_per_q) {
    if (index_per_q) return 1;
    if (group % 4 == 0) return 4;
    if (group % 2 == 0) return 2;
    return 1;
}

}  // namespace
