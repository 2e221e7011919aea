// Vertical-slash aggregation of the dense causal attention map (Sec. "Obtaining Ground Truth" of the paper) and
// Attention Recall of a vertical-slash mask (Eq. R(S)) for gfx950.
//
// The n x n probability matrix A = softmax(Q K^T / sqrt(d)) (causal) is never stored.  Two sweeps over the score tiles:
//   1. row sweep:    lse2[i] = log2 sum_j 2^(c s_ij), c = scale * log2(e): the normaliser of every row
//   2. column sweep: A[i,j] = 2^(c s_ij - lse2[i]) is recomputed tile by tile and added to its column sum A_v[j], to its
//                    diagonal sum A_s[i-j] and, where the mask keeps (i,j), to the recall.
// Both sweeps are the same kernel with the operands exchanged.  A workgroup (4 wavefronts) keeps 256 rows of the
// RESIDENT operand in registers (two blocks of 32 rows per wavefront, as the B operand of v_mfma_f32_32x32x16_bf16) and
// streams 32-row tiles of the other operand through LDS (A operand).  A lane then holds the scores of ONE resident row
// against 16 streamed rows, so the reduction over the streamed index is in-lane:
//   row sweep:    resident = queries, streamed = keys 0 .. diagonal  -> per-lane online max / sum over keys
//   column sweep: resident = keys,    streamed = queries diagonal .. n-1 -> per-lane sum over queries = column sum, kept
//                 in a register for the whole sweep; one store (one atomic where several workgroups or heads share a column).
// Two workgroups (row sweep: three) share a compute unit, so that one wavefront's matrix instructions run under the others' vector work.
// What bounds both sweeps is the vector work per score: scale and subtract, exponential (a quarter of the rate), add; the
// column sweep also adds every probability to its diagonal.
//
// The streamed rows are staged in an order that makes register e of a lane row 16 hh + e of the tile.
//
// Diagonal sums: element (streamed row r, resident key k) of a tile belongs to offset o = (first row - first key) + r - k.
// Tile (t, block c + 1) and tile (t - 1, block c) of a wavefront's two blocks hold the same offsets in the same places:
// they are added element by element first, and the diagonals are taken once for the two.  There, with k = 16 kh + l, register
// e moved e lanes down inside its row of 16 lanes (an operand modifier of the add) puts an element into the lane of its
// offset, 16 hh - 16 kh - l (d0), or, moved out at the lower end and in again at the upper, at 16 more (d1): 31 adds.  Of
// d1, the lanes of kh = 1 belong to the offsets of d0's lanes of kh = 0, those of kh = 0 to the offsets of the NEXT tile's d0
// lanes of kh = 1.  So every offset a half wavefront meets is finished in one place, once, and is stored, without a
// read or an atomic, to a 512-entry LDS ring that the half owns, indexed by o mod 512.  The offsets a workgroup can still touch
// form a window of 319 consecutive values that advances by 64 per stage; the 64 that fall out of it are added over the eight
// rings and flushed to global memory (one atomic each) every stage.
// (n = 16384, 32 / 8 heads with recall: 4.2 ms with one resident block per wavefront, a permutation through the LDS crossbar,
// two adds per element and LDS float atomics; 2.2 ms with all this but the atomics, two per pair of tiles, whose rate was
// the limit; now 1.23.  Row sweep 1.9 -> 0.96 ms.)
// Recall: a tile that no selected offset crosses adds its column sums where the column is selected; only crossed tiles look
// at single elements.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "vs_attn_device.h"
#include "vs_common.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kGroupRows = 64 * kWaves;        // resident rows per workgroup
constexpr int kStages = 2;                     // stages of two streamed tiles: one being read, one in flight
constexpr int kNormOff = kStages * 2 * kTileBytes;          // per streamed row of a stage: minus its normaliser (column sweep)
constexpr int kDiagRing = 512;                 // residues of an offset ring
constexpr int kDiagPitch = kDiagRing + 16;     // words from one ring to the next: the halves' offsets are 16 apart, their banks 32
constexpr int kRings = 2 * kWaves;             // one per half wavefront
constexpr int kDiagOff = kNormOff + kStages * 64 * 4;
constexpr float kLagSum = 512.f;               // entries of a row sweep up to 2^9 above the running maximum: their exponents are as exact as those below it
constexpr float kBelowMax = 1.f;               // the running maximum stays this far below: exponents of the entries that matter are smaller, and more exact
constexpr int kSmemBytes = kDiagOff + kRings * kDiagPitch * 4;

struct SweepParams {
    const uint16_t* q;              // [q_heads, n, 128]
    const uint16_t* k;              // [kv_heads, n, 128]
    float* lse2;                    // [q_heads, n]: row normalisers in the log2 domain, written by the row sweep
    const float* lse;               // what the column sweep reads: lse2, or the caller's natural-log normalisers
    float lse_scale;                // to the log2 domain
    float* a_v;                     // [out_heads, n], zeroed before the column sweep
    float* a_s;
    float* recall;                  // [out_heads] or null
    int q_heads, kv_heads, group, n;
    int reduce_group;               // 1: outputs are per KV head (mean over the group's query heads)
    float c;                        // scale * log2(e)
    float norm;                     // 1 / n (1 / (n group) when reducing), applied to the finished sums
    double* recall_acc;             // PARTS: per output head, the recall's sum and the workgroups that have added to it (zero at launch)
    unsigned int* recall_count;
    unsigned int recall_shares;     // PARTS: workgroups per output head
    const uint32_t* sbit;           // recall only; per index head: bit (o + 64) set iff offset o selected
    const uint32_t* vbit;           // recall only; per index head: bit j set iff column j selected
    int sw, vw, index_per_q;
    int parts;                      // PARTS: workgroups that share the streamed rows of one group of resident rows
    float2* row_part;               // row sweep with PARTS: [parts][q_heads, n] (maximum, sum) of a part's keys
    double* acc_v;                  // column sweep with PARTS: sums of a_v and a_s, [out_heads, n] each, zero at launch
    double* acc_s;
};

// x moved down by S lanes (row_shl) or up by S lanes (row_shr) inside every row of 16 lanes; lanes without a source get 0
template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

// One workgroup's share of a recall, one thread.  The shares of the shared-out form are many (up to 1024 for a single head: 4096
// float atomics of its wavefronts were off by 9e-7 at n = 16000), so they are added in fp64; who adds the last writes the recall.
__device__ __forceinline__ void add_recall_share(const SweepParams& p, int out_head, float share) {
    unsafeAtomicAdd(p.recall_acc + out_head, static_cast<double>(share));
    const unsigned int before = __hip_atomic_fetch_add(p.recall_count + out_head, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (before + 1u == p.recall_shares)
        p.recall[out_head] = static_cast<float>(__hip_atomic_load(p.recall_acc + out_head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) *
                                                static_cast<double>(p.norm));
}

// log2 of 2^m l.  The logarithm of the mantissa alone: it is rounded towards zero, by more the larger it is, and with a maximum that
// lags by up to 2^8 the sums are large (as m + log2(l) every row's entries came out 1.5e-7 too large, now below 3e-8).
__device__ __forceinline__ float normaliser(float m, float l) {
    const float base = m + static_cast<float>(__builtin_amdgcn_frexp_expf(l));
    return base + __log2f(__builtin_amdgcn_frexp_mantf(l));
}

// The parts of the shared-out row sweep: normaliser of every row (key 0 is causal for all: the sum is positive).
__global__ __launch_bounds__(kThreads) void combine_rows_kernel(const float2* __restrict__ part, int parts, int rows, float* __restrict__ lse2) {
    const int row = blockIdx.x * kThreads + threadIdx.x;
    if (row >= rows) return;
    float m = -INFINITY;
    for (int i = 0; i < parts; ++i) m = fmaxf(m, part[static_cast<size_t>(i) * rows + row].x);
    float l = 0.f;
    for (int i = 0; i < parts; ++i) {
        const float2 x = part[static_cast<size_t>(i) * rows + row];
        l += x.y * (x.x > -INFINITY ? __builtin_amdgcn_exp2f(x.x - m) : 0.f);   // the sum of a part with nothing but NaN is NaN
    }
    lse2[row] = normaliser(m, l);
}

// The sums of the shared-out column sweep.
__global__ __launch_bounds__(kThreads) void finish_sums_kernel(const double* __restrict__ acc_v, const double* __restrict__ acc_s, size_t count,
                                                               double norm, float* __restrict__ a_v, float* __restrict__ a_s) {
    const size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= count) return;
    a_v[i] = static_cast<float>(acc_v[i] * norm);
    a_s[i] = static_cast<float>(acc_s[i] * norm);
}

// COLUMNS == false: row sweep (resident queries, streamed keys).  COLUMNS == true: column sweep.
// PARTS: p.parts workgroups share the streamed rows of a group (a form of its own: the long sweeps lose 2 % with it).
// NB: resident blocks per wavefront; 1 (row sweep only) gives twice the workgroups of half the length when they are few and short.
template <bool COLUMNS, bool RECALL, bool PARTS = false, int NB = 2>
__global__ __launch_bounds__(kThreads, 2) void vs_sweep_kernel(const SweepParams p) {
    __shared__ __align__(16) unsigned char smem[kSmemBytes];
    float* const norm_ring = reinterpret_cast<float*>(smem + kNormOff);
    float* const diag = reinterpret_cast<float*>(smem + kDiagOff);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31, hh = lane >> 5;
    const int n = p.n;
    const float NEG_INF = -INFINITY;

    // ---- which 256 resident rows of which query head (and which part of the streamed rows); longest sweeps first ----
    const int h = blockIdx.x % p.q_heads;
    static_assert(NB == 2 || !COLUMNS, "the diagonal sums need both blocks");
    constexpr int kRows = 32 * NB * kWaves;                  // resident rows of this workgroup
    const int ngroups = (n + kRows - 1) / kRows;
    const int unit = blockIdx.x / p.q_heads;
    const int in_order = PARTS ? unit / p.parts : unit;
    const int grp = COLUMNS ? in_order : ngroups - 1 - in_order;
    const int g = h / p.group;
    const int out_head = p.reduce_group ? g : h;
    const int r0_wg = kRows * grp;
    const int my_r0 = r0_wg + 32 * NB * wave;                // rows my_r0 .. + 31 (block 0) and my_r0 + 32 .. + 63 (block 1)
    const int my_b0 = my_r0 >> 5;
    const uint16_t* __restrict__ res_base = COLUMNS ? p.k + static_cast<size_t>(g) * n * kD : p.q + static_cast<size_t>(h) * n * kD;
    const uint16_t* __restrict__ str_base = COLUMNS ? p.q + static_cast<size_t>(h) * n * kD : p.k + static_cast<size_t>(g) * n * kD;

    // ---- resident fragments: B operand; lane holds resident row qi, d = 16 kk + 8 hh .. +7 ----
    bf16x8 rf[NB][8];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint16_t* src = res_base + static_cast<size_t>(min(my_r0 + 32 * b + qi, n - 1)) * kD + 8 * hh;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) rf[b][kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + 16 * kk));
    }

    // ---- streamed tiles: keys 0 .. last resident row (rows), queries first resident row .. n-1 (columns) ----
    int t_begin = COLUMNS ? r0_wg >> 5 : 0;
    int t_end = COLUMNS ? (n + 31) >> 5 : (min(r0_wg + kRows, n) + 31) >> 5;
    int o_begin = 0;                                         // offset of the first streamed row to the first resident one
    if (PARTS) {
        // whole stages per part, as equal as they come; what the parts add up meets in the workspace
        const int part = unit % p.parts, stages = (t_end - t_begin + 1) >> 1;
        const int t0 = t_begin;
        t_begin = t0 + 2 * static_cast<int>(static_cast<long long>(stages) * part / p.parts);
        t_end = min(t_end, t0 + 2 * static_cast<int>(static_cast<long long>(stages) * (part + 1) / p.parts));
        if (t_begin >= t_end) {
            if (RECALL && tid == 0) add_recall_share(p, out_head, 0.f);
            if (!COLUMNS && r0_wg + tid < n)
                p.row_part[(static_cast<size_t>(part) * p.q_heads + h) * n + r0_wg + tid] = make_float2(NEG_INF, 0.f);
            return;
        }
        o_begin = 32 * (t_begin - t0);
    }
    const int nstages = (t_end - t_begin + 1) >> 1;

    if (COLUMNS) {
        for (int s = tid; s < kRings * kDiagPitch; s += kThreads) diag[s] = 0.f;
    }

    // recall: the resident key of this lane is a selected column -> every causal entry of the column is kept
    const int ih = p.index_per_q ? h : g;
    uint32_t col_keep[2] = {0u, 0u};
    const uint32_t* __restrict__ sbit = nullptr;
    if (RECALL) {
        sbit = p.sbit + static_cast<size_t>(ih) * p.sw;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int key = my_r0 + 32 * b + qi;
            if (key < n && ((p.vbit[static_cast<size_t>(ih) * p.vw + (key >> 5)] >> (key & 31)) & 1u)) col_keep[b] = 0xffffffffu;
        }
    }

    // ---- staging (the K layout of the attention kernels): wavefront w fills groups w and w + 4 of a tile, i.e. slots
    //      4 w + L / 16 and 16 more; slot 8 a + 4 h + c, which the matrix instruction returns in element 4 a + c of half h, holds
    //      row 16 h + 4 a + c; rows that do not exist read the last one (masked, or their normaliser is infinite) ----
    const int st_row = 16 * (wave & 1) + 4 * (wave >> 1) + (lane >> 4);
    const uint32_t st_b = static_cast<uint32_t>(16 * (4 * ((lane >> 2) & 3) + (((lane & 3) - (lane >> 4)) & 3)));
    // Requested with a stage and used one step later: used at once, they would be waited for together with the stage's rows
    // (memory requests return in order).
    float nreg = 0.f;                                        // normaliser of streamed row `tid` of the stage
    uint32_t wreg[3] = {0u, 0u, 0u};                         // offset bitmap from bit 32 (first tile - my block 0) + 32
    auto load_stage = [&](int st) __attribute__((always_inline)) {
        const int row0 = 32 * (t_begin + 2 * st);
        if (COLUMNS && tid < 64) nreg = p.lse[static_cast<size_t>(h) * n + min(row0 + tid, n - 1)];
        if (RECALL) {
            const uint32_t* const at = sbit + max(t_begin + 2 * st - my_b0, 0) + 1;
#pragma unroll
            for (int i = 0; i < 3; ++i) wreg[i] = at[i];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const int row = min(row0 + 32 * u + 8 * x + st_row, n - 1);
                lds_load16s((static_cast<uint32_t>(row) << 8) + st_b, str_base,
                            smem + (2 * (st & 1) + u) * kTileBytes + (wave + kWaves * x) * kGroupBytes);
            }
    };
    // A fragment kk: chunk 2 kk + hh of slot qi
    const int a_row = (qi >> 2) * kGroupBytes + (qi & 3) * 256;
    const int a_off0 = a_row + 16 * ((hh + qi) & 3), a_off2 = a_row + 16 * ((hh + qi + 2) & 3);

    auto read_a = [&](const unsigned char* at, int kk) __attribute__((always_inline)) -> bf16x8 {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(at + ((kk & 1) ? a_off2 : a_off0) + 64 * (kk >> 1)));
    };

    // ---- per-lane state ----
    float m_run[2] = {NEG_INF, NEG_INF}, l_run[2] = {0.f, 0.f};   // row sweep: running max (log2 domain) and sum of this lane's keys
    bool settled = false;                                         // every lane has a maximum (NB blocks; stays true)
    float col_sum[2] = {0.f, 0.f}, rec_sum = 0.f;                 // column sweep
    double col_total[2] = {0., 0.};                               // PARTS: col_sum moves here every four stages (5e-8 off instead of 8e-8 at n = 3000, three parts)
    f32x16 pend;                                             // column sweep: block 0's entries of the previous tile
#pragma unroll
    for (int e = 0; e < 16; ++e) pend[e] = 0.f;
    const int diag_lane = 16 * hh - (lane & 31);
    float* const my_diag = diag + kDiagPitch * (2 * wave + hh);
    const bool kh = (lane & 16) != 0;
    float d1_prev = 0.f;                                     // kh = 1: d1 of the previous tile's lanes of kh = 0
    uint64_t win_prev = 0ull;                                // block 0's window of the previous tile = block 1's of this one
    if (PARTS && RECALL && t_begin > my_b0) {
        const uint32_t* const at = sbit + (t_begin - my_b0);
        win_prev = uniform64(((static_cast<uint64_t>(at[1]) << 32) | at[0]) >> 1);
    }

    auto add_offset = [&](int o, float v) __attribute__((always_inline)) {
        const size_t at = static_cast<size_t>(out_head) * n + o;
        if constexpr (PARTS) unsafeAtomicAdd(p.acc_s + at, static_cast<double>(v));
        else unsafeAtomicAdd(p.a_s + at, v * p.norm);
    };

    // diagonals of one 32 x 32 set of entries; base: first row - first key.  Two chains each for d0 and d1.  Written out: from the builtin
    // the compiler makes 14 of the 30 moves instructions of their own.  (The wait covers the two states between a register's
    // write and its use through a lane move.)
    auto diagonals = [&](const f32x16& x, int base) __attribute__((always_inline)) {
        float d0[2], d1[2];
#define VS_DIAG(d, s, m) "v_add_f32_dpp %" #d ", %" #s ", %" #d " " m " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
#define VS_DIAG_FIRST(d, s, m) "v_mov_b32_dpp %" #d ", %" #s " " m " row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        asm("s_nop 1\n\t"
            "v_add_f32_dpp %0, %6, %4 row_shl:2 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
            VS_DIAG_FIRST(1, 5, "row_shl:1") VS_DIAG_FIRST(2, 6, "row_shr:14") VS_DIAG_FIRST(3, 5, "row_shr:15")
            VS_DIAG(0, 8, "row_shl:4") VS_DIAG(1, 7, "row_shl:3") VS_DIAG(2, 8, "row_shr:12") VS_DIAG(3, 7, "row_shr:13")
            VS_DIAG(0, 10, "row_shl:6") VS_DIAG(1, 9, "row_shl:5") VS_DIAG(2, 10, "row_shr:10") VS_DIAG(3, 9, "row_shr:11")
            VS_DIAG(0, 12, "row_shl:8") VS_DIAG(1, 11, "row_shl:7") VS_DIAG(2, 12, "row_shr:8") VS_DIAG(3, 11, "row_shr:9")
            VS_DIAG(0, 14, "row_shl:10") VS_DIAG(1, 13, "row_shl:9") VS_DIAG(2, 14, "row_shr:6") VS_DIAG(3, 13, "row_shr:7")
            VS_DIAG(0, 16, "row_shl:12") VS_DIAG(1, 15, "row_shl:11") VS_DIAG(2, 16, "row_shr:4") VS_DIAG(3, 15, "row_shr:5")
            VS_DIAG(0, 18, "row_shl:14") VS_DIAG(1, 17, "row_shl:13") VS_DIAG(2, 18, "row_shr:2") VS_DIAG(3, 17, "row_shr:3")
            VS_DIAG(1, 19, "row_shl:15") VS_DIAG(3, 19, "row_shr:1")
            : "=&v"(d0[0]), "=&v"(d0[1]), "=&v"(d1[0]), "=&v"(d1[1])
            : "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(x[6]), "v"(x[7]), "v"(x[8]), "v"(x[9]), "v"(x[10]), "v"(x[11]),
              "v"(x[12]), "v"(x[13]), "v"(x[14]), "v"(x[15]));
#undef VS_DIAG
#undef VS_DIAG_FIRST
        const float e1 = d1[0] + d1[1];
        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(e1), __float_as_uint(e1), false, false);
        const unsigned low = sw[0], high = sw[1];            // the values of kh = 0 / kh = 1 in all lanes
        my_diag[(base + diag_lane) & (kDiagRing - 1)] = (d0[0] + d0[1]) + (kh ? d1_prev : __uint_as_float(high));
        d1_prev = __uint_as_float(low);
    };

    // recall of a block's entries of a tile; sum: theirs; win: the tile's offset window
    auto add_recall = [&](const f32x16& x, float sum, uint64_t win, uint32_t col) __attribute__((always_inline)) {
        float rsum = __uint_as_float(__float_as_uint(sum) & col);
        if (win != 0ull) {
            const uint32_t keep = static_cast<uint32_t>(win >> (31 - qi + 16 * hh)) | col;   // bit e: (i, j) kept
            rsum = 0.f;
            static_for<16>([&](auto e_tag) __attribute__((always_inline)) {
                constexpr int e = decltype(e_tag)::value;
                uint32_t m;                                  // the keep-bit spread over a word
                asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(keep), "n"(e));
                rsum += __uint_as_float(__float_as_uint(x[e]) & m);
            });
        }
        rec_sum += rsum;
    };

    // Streamed tile t in slot `slot` against both resident blocks.  acc element e of lane (qi, hh) is (streamed row 16 hh +
    // e, resident row qi).  MASKED: the tile may hold entries past the diagonal.
    auto tile = [&](int t, int slot, uint32_t w0, uint32_t w1, auto masked_tag) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        const unsigned char* const at = smem + slot * kTileBytes;
        f32x16 acc[NB];
        {
            bf16x8 af[8];
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) af[kk] = read_a(at, kk);
            f32x16 zero;
#pragma unroll
            for (int e = 0; e < 16; ++e) zero[e] = 0.f;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                acc[0] = mfma32(af[kk], rf[0][kk], kk == 0 ? zero : acc[0]);
                if constexpr (NB == 2) acc[1] = mfma32(af[kk], rf[1][kk], kk == 0 ? zero : acc[1]);
            }
        }
        const int s0 = 32 * t;                               // first streamed row of the tile
        if constexpr (!COLUMNS) {
            // keys s0 .. s0+31 against queries: causal where key <= query
            if constexpr (!MASKED) {
                // The maxima as they stand, if no entry is more than 2^8 above its row's (the sums say so; not true for NaN); else the
                // tile is taken again and moves them, each time, or entries a little above would send every tile there.  (Maximum of every tile,
                // moved beyond 2^8: 32 / 8 heads, n = 16384 1.02 ms, now 0.96; n = 131072 55 vector instructions a tile beside matrix and exponentials, now 41.  Matrix
                // instructions issued between the exponentials, as in the column sweep: 1.00, three wavefronts share a SIMD here.)
                if (settled) {
                    float sum[NB][2];
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const float pr = __builtin_amdgcn_exp2f(fmaf(acc[b][e], p.c, -m_run[b]));
                            sum[b][e & 1] = e < 2 ? pr : sum[b][e & 1] + pr;
                        }
                    float worst = 0.f;
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        sum[b][0] += sum[b][1];
                        worst += sum[b][0];
                    }
                    if (!__ballot(!(worst < kLagSum))) {
#pragma unroll
                        for (int b = 0; b < NB; ++b) l_run[b] += sum[b][0];
                        return;
                    }
                }
            }
            settled = true;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                f32x16& x = acc[b];
                if constexpr (MASKED) {
                    const int lim = my_r0 + 32 * b + qi - s0 - 16 * hh;   // element e is causal iff e <= lim
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (e > lim) x[e] = NEG_INF;
                }
                float mt = fmaxf(fmaxf(x[0], x[1]), x[2]);
#pragma unroll
                for (int e = 3; e < 15; e += 2) mt = fmaxf(fmaxf(mt, x[e]), x[e + 1]);
                mt = fmaf(fmaxf(mt, x[15]), p.c, -kBelowMax);
                if (__ballot(mt > m_run[b])) {
                    const float m_new = fmaxf(m_run[b], mt);
                    l_run[b] *= m_new == NEG_INF ? 1.f : __builtin_amdgcn_exp2f(m_run[b] - m_new);
                    m_run[b] = m_new;
                }
                const float mc = m_run[b] == NEG_INF ? 0.f : m_run[b];
                float sum[2] = {0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 16; ++e) sum[e & 1] += __builtin_amdgcn_exp2f(fmaf(x[e], p.c, -mc));
                l_run[b] += sum[0] + sum[1];
                settled &= !__ballot(m_run[b] == NEG_INF);
            }
        } else {
            // queries s0 .. s0+31 against keys: causal where query >= key
            const float* const nr = norm_ring + 32 * slot + 16 * hh;
            f32x4 nv[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) nv[a] = *reinterpret_cast<const f32x4*>(nr + 4 * a);
            uint64_t win[2] = {0ull, 0ull};
            if (RECALL) {
                // selected offsets dlt-31 .. dlt+31 of a tile at bits 0..62, dlt = first query - first key
                // (w0, w1: bits dlt - 32 .. dlt + 31)
                win[0] = ((static_cast<uint64_t>(w1) << 32) | w0) >> 1;
                win[1] = win_prev;
                win_prev = win[0];
            }
            float psum[2];
#pragma unroll
            for (int b = 1; b >= 0; --b) {
                f32x16& x = acc[b];
                float sum[2];
                const int lim = my_r0 + 32 * b + qi - s0 - 16 * hh;       // element e is causal iff e >= lim
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float pr = __builtin_amdgcn_exp2f(fmaf(x[e], p.c, nv[e >> 2][e & 3]));
                    if (MASKED && e < lim) pr = 0.f;
                    x[e] = pr;
                    sum[e & 1] = e < 2 ? pr : sum[e & 1] + pr;
                    if (b == 1) pend[e] += pr;
                }
                psum[b] = sum[0] + sum[1];
                col_sum[b] += psum[b];
            }
            diagonals(pend, s0 - my_r0 - 32);
            pend = acc[0];
            if (RECALL) {
                add_recall(acc[0], psum[0], win[0], col_keep[0]);
                add_recall(acc[1], psum[1], win[1], col_keep[1]);
            }
        }
    };

    auto tile_any = [&](int t, int slot, uint32_t w0, uint32_t w1) __attribute__((always_inline)) {
        // live if any of its entries is causal for one of the two blocks
        const bool live = t < t_end && my_r0 < n && (COLUMNS ? t >= my_b0 : t <= my_b0 + NB - 1);
        if (!live) return;
        if (COLUMNS ? t <= my_b0 + 1 : t >= my_b0) tile(t, slot, w0, w1, std::true_type{});
        else tile(t, slot, w0, w1, std::false_type{});
    };

    // ---- column sweep: stages whose two tiles are whole for both blocks ----
    // The scores of a block are made between the vector instructions of the block before: slot (x, y) issues a matrix instruction for x,
    // then a piece of y, in a pipeline of its own (scale element pair k - 1, exponentials of k - 2, sums of k - 3: nothing waits for its
    // predecessor).  Two wavefronts share a SIMD, and one after the other they were in the same half of a tile too often.  Scheduling
    // barriers keep the order; arithmetic is pinned, or the compiler moves it to its use.  (32 / 8 heads, n = 16384 with recall 1.29 -> 1.26 ms with the
    // lane moves as operand modifiers, -> 1.23 with this.)
#define VS_PIN(x) asm volatile("" : "+v"(x))
    bf16x8 af[8];
    // MM: x = scores of the resident block with fragments rfb; the fragments af are replaced by those of the tile at `next` (if not null).
    // VV: y, scores -> entries 2^(c y + off(e)); sum: their sums, two chains; extra(k): more work for the pair k of entries
    auto slot = [&](auto mm, auto vv, const bf16x8 (&rfb)[8], f32x16& x, const unsigned char* next, f32x16& y, auto&& off, float (&sum)[2],
                    auto&& extra) __attribute__((always_inline)) {
        constexpr bool MM = decltype(mm)::value, VV = decltype(vv)::value;
        f32x16 zero;
#pragma unroll
        for (int e = 0; e < 16; ++e) zero[e] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
        static_for<VV ? 12 : 8>([&](auto k_tag) __attribute__((always_inline)) {
            constexpr int k = decltype(k_tag)::value;
            if constexpr (MM && k < 8) {
                x = mfma32(af[k], rfb[k], k == 0 ? zero : x);
                if (next) af[k] = read_a(next, k);
            }
            if constexpr (VV) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if constexpr (k >= 1 && k < 9) {
                        float t = fmaf(y[2 * (k - 1) + i], p.c, off(2 * (k - 1) + i));
                        VS_PIN(t);
                        y[2 * (k - 1) + i] = t;
                    }
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if constexpr (k >= 2 && k < 10) {
                        float t = __builtin_amdgcn_exp2f(y[2 * (k - 2) + i]);
                        VS_PIN(t);
                        y[2 * (k - 2) + i] = t;
                    }
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if constexpr (k >= 3 && k < 11) {
                        sum[i] = k == 3 ? y[2 * (k - 3) + i] : sum[i] + y[2 * (k - 3) + i];
                        VS_PIN(sum[i]);
                    }
                }
                if constexpr (k >= 3 && k < 11) extra(std::integral_constant<int, k - 3>{});
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    auto nothing = [](auto) __attribute__((always_inline)) {};
    // Column sweep, queries of stage st, t0: its first tile; w: words of the offset bitmap
    auto full_columns = [&](int st, int t0, const uint32_t (&w)[3]) __attribute__((always_inline)) {
        const unsigned char* const at = smem + 2 * (st & 1) * kTileBytes;
        const float* const nr = norm_ring + 64 * (st & 1) + 16 * hh;
        f32x16 x0, x1;
        f32x4 nv[4];
        float s[2];
        auto norms = [&](int u) __attribute__((always_inline)) {
#pragma unroll
            for (int a = 0; a < 4; ++a) nv[a] = *reinterpret_cast<const f32x4*>(nr + 32 * u + 4 * a);
        };
        auto off = [&](int e) __attribute__((always_inline)) { return nv[e >> 2][e & 3]; };
        auto into_pend = [&](auto k_tag) __attribute__((always_inline)) {
            constexpr int k = decltype(k_tag)::value;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float t = pend[2 * k + i] + x1[2 * k + i];
                VS_PIN(t);
                pend[2 * k + i] = t;
            }
        };
        auto through = [&](const f32x16& x, int b, uint64_t win) __attribute__((always_inline)) {
            const float sum = s[0] + s[1];
            col_sum[b] += sum;
            if (RECALL) add_recall(x, sum, win, col_keep[b]);
        };
        uint64_t win[2] = {0ull, 0ull};
        if (RECALL) {
            win[0] = ((static_cast<uint64_t>(w[1]) << 32) | w[0]) >> 1;
            win[1] = ((static_cast<uint64_t>(w[2]) << 32) | w[1]) >> 1;
        }
        norms(0);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) af[kk] = read_a(at, kk);
        slot(yes, no, rf[NB - 1], x1, nullptr, x1, off, s, nothing);
        slot(yes, yes, rf[0], x0, at + kTileBytes, x1, off, s, into_pend);
        through(x1, 1, win_prev);
        diagonals(pend, 32 * t0 - my_r0 - 32);
        slot(yes, yes, rf[NB - 1], x1, nullptr, x0, off, s, nothing);
        pend = x0;
        through(pend, 0, win[0]);
        norms(1);
        slot(yes, yes, rf[0], x0, nullptr, x1, off, s, into_pend);
        through(x1, 1, win[0]);
        diagonals(pend, 32 * t0 - my_r0);
        slot(no, yes, rf[0], x1, nullptr, x0, off, s, nothing);
        pend = x0;
        through(pend, 0, win[1]);
        win_prev = win[1];
    };
#undef VS_PIN

    // ---- pipeline: step s computes stage s; the loads of stage s + 1 are issued at its top, over stage s - 1 ----
    load_stage(0);
    for (int st = 0; st < nstages; ++st) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // this wavefront's part of stage st (and the resident rows) has arrived
        if (COLUMNS && tid < 64) {
            // 2^(c s - lse2) is the entry of A; rows that do not exist get 2^-inf
            const bool exists = 32 * (t_begin + 2 * st) + tid < n;
            norm_ring[64 * (st & 1) + tid] = exists ? -(nreg * p.lse_scale) : NEG_INF;
        }
        uint32_t w[3] = {0u, 0u, 0u};
        if (RECALL) {
#pragma unroll
            for (int i = 0; i < 3; ++i) w[i] = __builtin_amdgcn_readfirstlane(wreg[i]);
        }
        __syncthreads();
        if (COLUMNS && st > 0) {
            // offsets below 64 st - 255 can no longer be touched: flush the 64 that became final with the last stage, 16 per
            // wavefront; a row of 16 lanes adds two rings
            const int o = o_begin + 64 * (st - 1) - (kGroupRows - 1) + 16 * wave + (lane & 15);
            float* const at = diag + 2 * kDiagPitch * (lane >> 4) + (o & (kDiagRing - 1));
            float v = at[0] + at[kDiagPitch];
            at[0] = at[kDiagPitch] = 0.f;
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
            const unsigned low = sw[0], high = sw[1];
            v = half_swap_sum(__uint_as_float(low) + __uint_as_float(high));
            if (lane < 16 && o >= 0 && o < n && v != 0.f) add_offset(o, v);
        }
        if (st + 1 < nstages) load_stage(st + 1);
        const int t0 = t_begin + 2 * st;
        bool done = false;
        if constexpr (COLUMNS) {
            if (t0 > my_b0 + 1 && t0 + 1 < t_end && my_r0 < n) {
                full_columns(st, t0, w);
                done = true;
            }
        }
        if (!done) {
            tile_any(t0, 2 * (st & 1), w[0], w[1]);
            tile_any(t0 + 1, 2 * (st & 1) + 1, w[1], w[2]);
        }
        if constexpr (COLUMNS && PARTS) {
            if ((st & 3) == 3) {
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    col_total[b] += static_cast<double>(col_sum[b]);
                    col_sum[b] = 0.f;
                }
            }
        }
    }

    // ---- results ----
    if constexpr (!COLUMNS) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            // the two halves of the wavefront hold disjoint keys of the same query: merge (max, sum) pairs
            const auto mo = __builtin_amdgcn_permlane32_swap(__float_as_uint(m_run[b]), __float_as_uint(m_run[b]), false, false);
            const auto lo = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run[b]), __float_as_uint(l_run[b]), false, false);
            const float m_a = __uint_as_float(mo[0]), m_b = __uint_as_float(mo[1]);
            const float l_a = __uint_as_float(lo[0]), l_b = __uint_as_float(lo[1]);
            const float m2 = fmaxf(m_a, m_b);
            float l2 = 0.f;
            l2 += l_a * (m_a > NEG_INF ? __builtin_amdgcn_exp2f(m_a - m2) : 0.f);   // (a NaN sum stays NaN)
            l2 += l_b * (m_b > NEG_INF ? __builtin_amdgcn_exp2f(m_b - m2) : 0.f);
            const int row = my_r0 + 32 * b + qi;
            if constexpr (PARTS) {
                if (row < n && hh == 0)
                    p.row_part[(static_cast<size_t>(unit % p.parts) * p.q_heads + h) * n + row] = make_float2(m2, l2);
                continue;
            }
            if (row < n && hh == 0) p.lse2[static_cast<size_t>(h) * n + row] = normaliser(m2, l2);
        }
    } else {
        if (my_r0 < n && (!PARTS || my_b0 < t_end)) {
            // block 0's entries of the last tile have no partner; what they leave in d1_prev has no next tile
            const int base = 32 * (t_end - 1) - my_r0;
            diagonals(pend, base);
            my_diag[(base + 32 + diag_lane) & (kDiagRing - 1)] = kh ? d1_prev : 0.f;
        }
        __syncthreads();
        // what is still in the ring: the last 319 offsets the workgroup touched
        for (int i = tid; i < kGroupRows + 64; i += kThreads) {
            const int o = o_begin + 64 * (nstages - 1) - (kGroupRows - 1) + i;
            if (o >= 0 && o < n) {
                float v = 0.f;
#pragma unroll
                for (int r = 0; r < kRings; ++r) v += diag[r * kDiagPitch + (o & (kDiagRing - 1))];
                if (v != 0.f) add_offset(o, v);
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int key = my_r0 + 32 * b + qi;
            const size_t at = static_cast<size_t>(out_head) * n + key;
            if constexpr (PARTS) {
                // (both halves of the wavefront add)
                if (key < n) unsafeAtomicAdd(p.acc_v + at, col_total[b] + static_cast<double>(col_sum[b]));
            } else {
                const float cs = half_swap_sum(col_sum[b]);
                if (key < n && hh == 0) {
                    if (p.reduce_group) unsafeAtomicAdd(p.a_v + at, cs * p.norm);
                    else p.a_v[at] = cs * p.norm;
                }
            }
        }
        if (RECALL) {
            float r = rec_sum;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) r += __shfl_xor(r, d);
            if constexpr (PARTS) {
                if (lane == 0) norm_ring[wave] = r;          // (idle since the barrier above)
                __syncthreads();
                if (tid == 0) add_recall_share(p, out_head, (norm_ring[0] + norm_ring[1]) + (norm_ring[2] + norm_ring[3]));
            } else {
                if (lane == 0 && r != 0.f) unsafeAtomicAdd(p.recall + out_head, r * p.norm);
            }
        }
    }
}

// Everything a call starts from, in one launch: the bitmaps of the mask's lists (a workgroup each, built in LDS and written out whole),
// zeroed outputs and sums.  (Clearing the bitmaps and setting their bits with global atomics were three launches: with recall, one head,
// n = 1000 38 -> 31 us, 8 / 2 heads, n = 1500 42 -> 35, 32 / 8 heads, n = 2000 83 -> 80.)
constexpr int kSetupThreads = 1024;
struct SetupParams {
    const int32_t* idx[2];          // offsets, columns
    const int32_t* cnt[2];
    int cap[2];
    uint32_t* bits[2];              // per index head: words[.] words, bit e + shift[.] for every list entry e
    int words[2], shift[2];
    int n, index_heads;             // index_heads: 0 without a mask
    float* a_v;                     // outputs that are accumulated in place
    float* a_s;
    size_t count;
    float* recall;
    int heads;
    uint32_t* sums;                 // workspace words
    size_t sum_words;
};

__global__ __launch_bounds__(kSetupThreads) void setup_kernel(const SetupParams p) {
    extern __shared__ uint32_t bm[];
    const int tid = threadIdx.x, block = blockIdx.x;
    if (block < 2 * p.index_heads) {
        const int list = block & 1, ih = block >> 1, words = p.words[list];
        for (int w = tid; w < words; w += kSetupThreads) bm[w] = 0u;
        __syncthreads();
        const int m = min(p.cnt[list][ih], p.cap[list]);
        for (int t = tid; t < m; t += kSetupThreads) {
            const int e = p.idx[list][static_cast<size_t>(ih) * p.cap[list] + t];
            const int bit = e + p.shift[list];
            if (e >= 0 && e < p.n) atomicOr(&bm[bit >> 5], 1u << (bit & 31));
        }
        __syncthreads();
        uint32_t* const out = p.bits[list] + static_cast<size_t>(ih) * words;
        for (int w = tid; w < words; w += kSetupThreads) out[w] = bm[w];
        return;
    }
    const size_t i = static_cast<size_t>(block - 2 * p.index_heads) * kSetupThreads + tid;
    if (i < p.count) {
        p.a_v[i] = 0.f;
        p.a_s[i] = 0.f;
    }
    if (p.recall && i < static_cast<size_t>(p.heads)) p.recall[i] = 0.f;
    if (i < p.sum_words) p.sums[i] = 0u;
}

// Up to 1024 groups of resident rows (512 workgroups run at once, and the longest sweep is twice the average): the streamed rows of a
// group are shared out over several workgroups of at least four stages of two tiles; their column and diagonal sums are added in fp64 (as
// float atomics the sums of more, shorter parts were up to twice as far off).  About 600 workgroups in all, up to 1024 where a part still has
// sixteen stages: a part has an end of its own (up to 319 offsets and 256 columns to add, the recall's share), and the workgroups wait for
// each other's.  us per call with recall, not shared / shared, and with how many parts: one head, n = 4000 (16 groups, 63 stages) 217 / 38 (16), 8000
// (32, 125) 414 / 57 (16; with 32 79), 16000 (63, 250) 802 / 119 (12; 16 121); 4 heads, n = 3192 (52, 50) 178 / 54 (11; 13 57); 8 / 2 heads, n = 2867
// (96, 45) 161 / 52 (6; 10 62), 5000 (160, 79) 270 / 98 (4; 3 118), 8000 (256, 125) 423 / 192 (4; 2 249); 32 / 8 heads, n = 1000 (128, 16) 67 / 39 (4),
// 1500 (192, 24) 94 / 57 (3; 5 64), 4000 (512, 63) 234 / 196 (2), 8192 (1024, 128) 663 / 642 (2); 64 / 8 heads, n = 1400 (384, 22) 91 / 80 (2),
// 2837 (768, 45) 194 / 218 (2; the fp64 sums are worth it, 7.6e-8 off instead of 1.25e-7).
int sweep_parts(int q_heads, int64_t n) {
    const int64_t groups = static_cast<int64_t>(q_heads) * ((n + kGroupRows - 1) / kGroupRows), stages = (n + 63) / 64;
    if (groups > 1024) return 1;
    const int64_t parts = std::max<int64_t>({2, 600 / groups, std::min(1024 / groups, stages / 16)});
    return static_cast<int>(std::min(parts, (stages + 3) / 4));
}

struct AggWs {
    size_t lse_off, sbit_off, vbit_off, acc_off, count_off, sums_off, row_off, total;
    int sw, vw;
};

AggWs agg_ws_layout(int q_heads, int index_heads, int64_t n) {
    AggWs w;
    w.sw = static_cast<int>(vs::round_up(static_cast<size_t>(n + 64 + 160 + 31) / 32, 4));
    w.vw = static_cast<int>(vs::round_up(static_cast<size_t>((n + 31) / 32 + 4), 4));
    w.lse_off = 0;
    w.sbit_off = vs::round_up(static_cast<size_t>(q_heads) * n * 4, 256);
    w.vbit_off = w.sbit_off + static_cast<size_t>(index_heads) * w.sw * 4;
    // (recall wanted: fp64 sums and arrival counts, zeroed at the start of a call)
    w.acc_off = vs::round_up(w.vbit_off + static_cast<size_t>(index_heads) * w.vw * 4, 8);
    w.count_off = w.acc_off + (index_heads > 0 ? static_cast<size_t>(q_heads) * 8 : 0);
    w.sums_off = vs::round_up(w.count_off + (index_heads > 0 ? static_cast<size_t>(q_heads) * 4 : 0), 256);
    const int parts = sweep_parts(q_heads, n);
    // shared-out sweeps: fp64 sums of a_v and a_s (zeroed as well), the row sweep's partial results
    w.row_off = w.sums_off + (parts > 1 ? vs::round_up(2 * static_cast<size_t>(q_heads) * n * sizeof(double), 256) : 0);
    w.total = w.row_off + (parts > 1 ? vs::round_up(static_cast<size_t>(parts) * q_heads * n * sizeof(float2), 256) : 0);
    return w;
}

}  // namespace

extern "C" {

size_t vs_aggregate_workspace(int q_heads, int kv_heads, int index_heads, int64_t n) {
    if (q_heads <= 0 || kv_heads <= 0 || index_heads < 0 || n <= 0 || n > VS_MAX_SEQ) return 0;
    // A workspace that is enough for n is enough for shorter sequences, also for those whose sweeps are shared out where those of n are not:
    // the largest of them, at the lengths where the number of parts can change.
    size_t most = agg_ws_layout(q_heads, index_heads, n).total;
    for (int64_t m = 64; m < n && q_heads * ((m + kGroupRows - 1) / kGroupRows) <= 1024; m += 64)
        most = std::max(most, agg_ws_layout(q_heads, index_heads, m).total);
    return most;
}

int vs_aggregate(const void* q, const void* k, int q_heads, int kv_heads, int64_t n, float scale, const float* lse,
                 int out_heads, float* a_v, float* a_s, const int32_t* idx_v, const int32_t* cnt_v, int cap_v,
                 const int32_t* idx_s, const int32_t* cnt_s, int cap_s, int index_heads, float* recall, void* ws,
                 size_t ws_bytes, void* stream) {
    if (!q || !k || !a_v || !a_s) return VS_ERR_INVALID_ARG;
    if (!vs::aligned16(q) || !vs::aligned16(k) || !vs::aligned16(a_v) || !vs::aligned16(a_s)) return VS_ERR_INVALID_ARG;
    if (q_heads <= 0 || kv_heads <= 0 || n <= 0) return VS_ERR_INVALID_ARG;
    if (!(scale > 0.f) || !isfinite(scale)) return VS_ERR_INVALID_ARG;
    if (q_heads % kv_heads != 0) return VS_ERR_UNSUPPORTED;
    if (n > VS_MAX_SEQ) return VS_ERR_UNSUPPORTED;
    if (out_heads != q_heads && out_heads != kv_heads) return VS_ERR_UNSUPPORTED;
    const bool want_recall = recall != nullptr;
    if (want_recall) {
        if (!idx_v || !cnt_v || !idx_s || !cnt_s || cap_v <= 0 || cap_s <= 0) return VS_ERR_INVALID_ARG;
        if (index_heads != kv_heads && index_heads != q_heads) return VS_ERR_UNSUPPORTED;
    } else {
        index_heads = 0;
    }
    const AggWs w = agg_ws_layout(q_heads, index_heads, n);
    if (!ws || ws_bytes < w.total) return VS_ERR_WORKSPACE;
    if (!vs::aligned16(ws)) return VS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char* base = static_cast<unsigned char*>(ws);

    SweepParams p{};
    p.parts = 1;
    p.q = static_cast<const uint16_t*>(q);
    p.k = static_cast<const uint16_t*>(k);
    p.lse2 = reinterpret_cast<float*>(base + w.lse_off);
    p.a_v = a_v;
    p.a_s = a_s;
    p.recall = recall;
    p.q_heads = q_heads;
    p.kv_heads = kv_heads;
    p.group = q_heads / kv_heads;
    p.n = static_cast<int>(n);
    p.reduce_group = (out_heads != q_heads) ? 1 : 0;
    p.c = scale * 1.4426950408889634f;
    p.norm = static_cast<float>(1.0 / (static_cast<double>(n) * (p.reduce_group ? p.group : 1)));
    p.index_per_q = (want_recall && index_heads == q_heads && q_heads != kv_heads) ? 1 : 0;

    const size_t out_count = static_cast<size_t>(out_heads) * n;
    const int parts = sweep_parts(q_heads, n);
    SetupParams sp{};
    sp.n = p.n;
    if (want_recall) {
        sp.index_heads = index_heads;
        sp.idx[0] = idx_s;
        sp.idx[1] = idx_v;
        sp.cnt[0] = cnt_s;
        sp.cnt[1] = cnt_v;
        sp.cap[0] = cap_s;
        sp.cap[1] = cap_v;
        sp.words[0] = p.sw = w.sw;
        sp.words[1] = p.vw = w.vw;
        sp.shift[0] = 64;
        sp.bits[0] = reinterpret_cast<uint32_t*>(base + w.sbit_off);
        sp.bits[1] = reinterpret_cast<uint32_t*>(base + w.vbit_off);
        p.sbit = sp.bits[0];
        p.vbit = sp.bits[1];
    }
    sp.a_v = a_v;
    sp.a_s = a_s;
    sp.count = parts > 1 ? 0 : out_count;
    sp.recall = recall;
    sp.heads = out_heads;
    sp.sums = reinterpret_cast<uint32_t*>(base + w.acc_off);
    sp.sum_words = (w.sums_off + (parts > 1 ? 2 * out_count * sizeof(double) : 0) - w.acc_off) / 4;
    size_t most = sp.count > sp.sum_words ? sp.count : sp.sum_words;
    if (most < static_cast<size_t>(out_heads)) most = out_heads;
    const size_t setup_lds = want_recall ? static_cast<size_t>(w.sw > w.vw ? w.sw : w.vw) * 4 : 0;
    const size_t setup_blocks = 2 * static_cast<size_t>(index_heads) + (most + kSetupThreads - 1) / kSetupThreads;
    if (setup_lds > 160 * 1024 || setup_blocks > 0x7fffffff) return VS_ERR_UNSUPPORTED;
    static vs::PerDeviceOnce once;
    const int rc = once.run(nullptr, [](int) -> int {
        VS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&setup_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
        return VS_OK;
    });
    if (rc != VS_OK) return rc;
    hipLaunchKernelGGL(setup_kernel, dim3(static_cast<unsigned>(setup_blocks)), dim3(kSetupThreads), setup_lds, st, sp);
    VS_LAUNCH_CHECK();
    const int64_t blocks = static_cast<int64_t>(q_heads) * ((n + kGroupRows - 1) / kGroupRows);
    if (blocks > 0x7fffffffLL) return VS_ERR_UNSUPPORTED;
    p.lse = lse ? lse : p.lse2;
    p.lse_scale = lse ? 1.4426950408889634f : 1.f;
    p.parts = parts;
    p.acc_v = reinterpret_cast<double*>(base + w.sums_off);
    p.acc_s = p.acc_v + out_count;
    p.row_part = reinterpret_cast<float2*>(base + w.row_off);
    const dim3 grid(static_cast<unsigned>(blocks * parts));
    if (!lse) {
        if (parts > 1) {
            hipLaunchKernelGGL((vs_sweep_kernel<false, false, true>), grid, dim3(kThreads), 0, st, p);
            VS_LAUNCH_CHECK();
            const int rows = q_heads * static_cast<int>(n);  // at most 1024 groups of 256
            hipLaunchKernelGGL(combine_rows_kernel, dim3(static_cast<unsigned>((rows + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                               p.row_part, parts, rows, p.lse2);
        } else if (n <= kGroupRows && blocks <= 256) {
            // One group per head, not shared out: workgroups of half a group, since the call lasts as long as one workgroup.  us per call, halves /
            // whole groups: one head, n = 200 17 / 20, 256 19 / 22, 128 heads, n = 200 18 / 22, 256 heads, n = 256 21 / 24; 512 heads 34 / 34, 1024
            // heads, n = 160 43 / 42.
            const int64_t halves = static_cast<int64_t>(q_heads) * ((n + kGroupRows / 2 - 1) / (kGroupRows / 2));
            hipLaunchKernelGGL((vs_sweep_kernel<false, false, false, 1>), dim3(static_cast<unsigned>(halves)), dim3(kThreads), 0, st, p);
        } else {
            hipLaunchKernelGGL((vs_sweep_kernel<false, false>), grid, dim3(kThreads), 0, st, p);
        }
        VS_LAUNCH_CHECK();
    }
    if (want_recall) {
        p.recall_acc = reinterpret_cast<double*>(base + w.acc_off);
        p.recall_count = reinterpret_cast<unsigned int*>(base + w.count_off);
        p.recall_shares = static_cast<unsigned int>(blocks / q_heads * parts * (p.reduce_group ? p.group : 1));
    }
    if (parts > 1) {
        if (want_recall) hipLaunchKernelGGL((vs_sweep_kernel<true, true, true>), grid, dim3(kThreads), 0, st, p);
        else hipLaunchKernelGGL((vs_sweep_kernel<true, false, true>), grid, dim3(kThreads), 0, st, p);
        VS_LAUNCH_CHECK();
        hipLaunchKernelGGL(finish_sums_kernel, dim3(static_cast<unsigned>((out_count + kThreads - 1) / kThreads)), dim3(kThreads), 0, st, p.acc_v,
                           p.acc_s, out_count, 1.0 / (static_cast<double>(n) * (p.reduce_group ? p.group : 1)), a_v, a_s);
    } else {
        if (want_recall) hipLaunchKernelGGL((vs_sweep_kernel<true, true>), grid, dim3(kThreads), 0, st, p);
        else hipLaunchKernelGGL((vs_sweep_kernel<true, false>), grid, dim3(kThreads), 0, st, p);
    }
    VS_LAUNCH_CHECK();
    return VS_OK;
}

}  // extern "C"
