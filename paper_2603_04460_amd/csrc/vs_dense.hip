// Dense causal attention for gfx950 on the layout of the sparse kernel (bf16 Q / K / V, head dimension 128, GQA).
//
// Four wavefronts per workgroup, one per SIMD, each owning TWO 32-row blocks of the workgroup's 8 (hc query heads of
// the KV group times 8 / hc consecutive 32-row sub-blocks).  Every K / V fragment read from LDS feeds two matrix
// instructions, one per row block, which halves the LDS reads per flop against one row block per wavefront.  The
// arithmetic per row block (S^T = K Q^T, joint softmax over a stage of two 32-key tiles with a lazily updated
// maximum, O^T = V^T P^T) and the LDS tile layout are those of the sparse kernel.
//
// One wavefront issues a vector instruction every 5.4 clocks (two on a SIMD one every 2.7; an exponential takes 8.8, and 8.3), while a 32x32x16
// matrix instruction occupies the matrix core for 32 and overlaps with what stands beside it: with five vector instructions and an exponential
// behind it 42 clocks from one wavefront, 39 from two (profiles/issue_rates.txt).  With one wavefront per SIMD nothing hides a wait, so the kernel is written to
// give every matrix instruction such company and nothing in a burst: the two row blocks run half a stage apart and each slot is written
// out in issue order, matrix and vector instructions, fragment reads and staging loads alternating.
//   slot X(i): matrix: scores of block 0 for stage i, then P V of block 0 for stage i-1;  vector: softmax of block 1, stage i-1
//   slot Y(i): matrix: scores of block 1 for stage i, then P V of block 1 for stage i-1;  vector: softmax of block 0, stage i
// V fragments of stage i-1 are read at the start of X(i), K fragments of stage i+1 in Y(i) after the scores of
// block 1; one barrier per stage, in Y(i), publishes stage i+1 and frees the buffer of stage i-1 for stage i+2.
//
// Stages below the diagonal but for the first take the row maximum as it stands (vs_attn_device.h, "stages without a row maximum"): with the
// search for it a tile had 94 vector instructions, now 77, and it held the exponentials back (32 / 8 heads x 8192 487 -> 458 us, x 16384 1857 -> 1737).
// The sum of a lane's weights is looked at in front of the last matrix instruction of their slot; where every stage moves the maximum (scores that
// grow by 2^1000 over 8192 keys) the call takes 590 us, 515 with the search in every stage.  Their V fragments are
// read one behind each score product (all within the first six of them the four wavefronts asked the LDS for three times what it
// gives) and their staging loads are issued between the score products of block 1 (all eight behind the barrier kept the matrix core
// waiting): 458 -> 435 and 1737 -> 1642 us; with all this the matrix core is busy 76 % of the cycles at 1.65 GHz (n = 131072; 60 % at 1.99 before: the
// chip's power, not the instruction stream, is what bounds it now).
// A row block behind the last position has no mask either: for it alone the others of its wavefront ran every stage with one
// (32 / 8 heads x 3152, half of the last workgroup's rows missing, 104 -> 79 us, x 1500 50 -> 37, 8 / 2 x 15000 485 -> 364).
//
// Built with -mllvm -amdgpu-mfma-vgpr-form: score accumulators are then written to the vector registers the softmax
// reads them from (the default puts every accumulator of a 512-register kernel in the accumulation registers and
// copies element by element).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "vs_attn_device.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr size_t kSmemBytes = kSlots * kSlotBytes;
constexpr size_t kDuoBytes = 2 * kWaves * kSlotBytes;
static_assert(kPartialBytes <= kDuoBytes && kDuoBytes <= 160 * 1024, "partial results in the idle buffers, one workgroup per compute unit");
// f(integral_constant<int, FROM>), .., f(integral_constant<int, TO - 1>)
template <int FROM, int TO, class F>
__device__ __forceinline__ void unroll(F f) {
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        unroll<FROM + 1, TO>(f);
    }
}

constexpr int kShortUnits = 128;               // workgroups up to which the keys of a row block are split
constexpr int kDuoKeys = 2048;

// DUO: few row blocks.  The workgroup has two row blocks, and every wavefront owns both; the keys are split over the wavefronts, which
// take stages of two tiles in turn, each through a K and a V buffer of its own that it fills itself (no barrier): stage i of
// wavefront w are the tiles 2 (4 i + w) and the next.  The fragments of a stage are read in the slot before their use, so a buffer can be
// filled again a whole slot before the next fragment is read from it.  Against vs_short_kernel (one row block per wavefront, tiles shared by two
// wavefronts), which is bound by the LDS (64 KB staged and 128 KB of fragments read for four tiles), half the fragments are read: 500 rows
// against 32768 keys, 32 / 8 heads, 322 -> 282 us, 300 rows 282 -> 214, one head of 16384 143 -> 111.
// Bound by matrix products and loads alike: 2048 clocks each for a stage of the four wavefronts (128 KB at 64 bytes a clock).  The loads go out one
// behind each matrix instruction, 46 of them before their data is needed (all of K in the X slot and of V in the Y slot, half a slot and
// a little more, had to wait), without address arithmetic: 270 -> 254 us, 1128 rows of 30575 keys 652 -> 597, one head of 16001 103 -> 93; the
// matrix core is busy 60 % of the cycles at 1.65 GHz (500 rows, profiles/cases_instruction_mix.txt).
template <bool DUO>
__global__ __launch_bounds__(kThreads) void vs_dense_kernel(const AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const kvbuf = smem;
    const float NEG_INF = -INFINITY;
    const int bid = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31, hh = lane >> 5;
    const int rest = bid / p.kv_heads;
    const int g = bid % p.kv_heads;
    const int hchunks = p.group / p.hc;
    const int hchunk = rest % hchunks;
    const int tile = p.tiles - 1 - rest / hchunks;          // longest tiles first
    const int BQ = (DUO ? 64 : 256) / p.hc;
    const int i0 = p.pos0 + tile * BQ;                      // positions are absolute; the tile grid starts at the chunk
    const int n = p.n;                                      // keys up to the last position (those behind it are not read)
    const int n_pos = p.pos0 + p.nq;                        // positions that exist
    const int i_last = min(i0 + BQ, n_pos) - 1;

    int my_head[2], my_i0[2];
    bool my_rows[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const int w = DUO ? rb : 2 * wave + rb;
        my_head[rb] = g * p.group + hchunk * p.hc + w % p.hc;
        my_i0[rb] = i0 + 32 * (w / p.hc);
        my_rows[rb] = my_i0[rb] < n_pos;
    }
    const uint16_t* __restrict__ kbase = p.k + static_cast<size_t>(g) * p.kv_rows * kD;
    const uint16_t* __restrict__ vbase = p.v + static_cast<size_t>(g) * p.kv_rows * kD;

    bf16x8 qf[2][8];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const int row = my_i0[rb] + qi;
        const uint16_t* src = p.q + (static_cast<size_t>(my_head[rb]) * p.nq + (min(row, n_pos - 1) - p.pos0)) * kD + 8 * hh;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            uint4 raw = make_uint4(0, 0, 0, 0);
            if (row < n_pos) raw = *reinterpret_cast<const uint4*>(src + 16 * kk);
            qf[rb][kk] = __builtin_bit_cast(bf16x8, raw);
        }
    }
    f32x16 oacc[2][4];
    float m_run[2], l_run[2];

    // staging: wavefront w fills groups w and w + 4 of a tile (rows 4 w + L / 16 and 16 more)
    const int st_row = tid >> 4;
    const int st_rho = (lane >> 4) & 3;
    const int st_ck = 4 * ((lane >> 2) & 3) + (((lane & 3) - st_rho) & 3);
    const int st_cv = 4 * ((((lane >> 2) & 3) - st_rho) & 3) + (lane & 3);
    const int nblk = i_last / 32 + 1;
    const int nst = DUO ? (nblk + 2 * kWaves - 1) / (2 * kWaves) : (nblk + 1) >> 1;
    // first tile of a stage, in units of two
    auto pair_of = [&](int st) __attribute__((always_inline)) { return DUO ? kWaves * st + wave : st; };
    // per-thread byte offsets of its four pieces of a stage (tile u, row half h), relative to the stage's first row
    uint32_t voff_k[2][2], voff_v[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            voff_k[u][h] = static_cast<uint32_t>(((32 * u + st_row + 16 * h) * kD + st_ck * 8) * 2);
            voff_v[u][h] = static_cast<uint32_t>(((32 * u + st_row + 16 * h) * kD + st_cv * 8) * 2);
        }
    // piece 0 .. 7 of this thread's share of a stage: (tile u, row half h) of K, then of V; whole: every row of the stage exists
    auto load_piece = [&](int st, int piece, bool whole) __attribute__((always_inline)) {
        const int u = piece >> 2, h = (piece >> 1) & 1, v = piece & 1;
        unsigned char* const dst = kvbuf + (2 * (st % 3) + u) * kSlotBytes + (wave + 4 * h) * kGroupBytes + v * kTileBytes;
        const uint16_t* const base = v ? vbase : kbase;
        if (whole) {
            // uniform base + per-thread offset, no address arithmetic per load
            lds_load16s(v ? voff_v[u][h] : voff_k[u][h], base + static_cast<size_t>(64 * st) * kD, dst);
            return;
        }
        const int t = 2 * st + u;
        int row = 32 * t + st_row + 16 * h;
        if (t >= nblk || row >= n) row = 0;                  // masked anyway: no predicate on the load (every row has key 0)
        lds_load16(base + static_cast<size_t>(row) * kD + (v ? st_cv : st_ck) * 8, dst);
    };
    auto whole_stage = [&](int st) __attribute__((always_inline)) { return 2 * st + 1 < nblk && 64 * st + 63 < n; };
    auto load_stage = [&](int st) __attribute__((always_inline)) {
        const bool whole = whole_stage(st);
#pragma unroll
        for (int piece = 0; piece < 8; ++piece) load_piece(st, piece, whole);
    };
    // DUO: one group of four rows of tile u of the wavefront's own stage, row (lane / 16) of it; row0: the tile's first row.  WHOLE: the tile
    // exists for the workgroup; otherwise rows behind the workgroup's last are masked and read that one.
    unsigned char* const own = kvbuf + wave * 2 * kSlotBytes;
    auto load_own = [&](auto whole, int v, int u, auto group, int row0) __attribute__((always_inline)) {
        constexpr int GRP = decltype(group)::value;
        const uint32_t chunk = static_cast<uint32_t>(v ? st_cv : st_ck) * 16u;
        unsigned char* const dst = own + u * kSlotBytes + v * kTileBytes + GRP * kGroupBytes;
        if constexpr (decltype(whole)::value) {
            const uint16_t* const rows = (v ? vbase : kbase) + static_cast<size_t>(row0 + 16 * (GRP / 4)) * kD;
            lds_load16o<1024 * (GRP % 4)>(static_cast<uint32_t>(st_rho) * 256u + chunk, rows, dst);
        } else {
            const uint32_t at = static_cast<uint32_t>(row0 + 4 * GRP + st_rho) * 256u;
            lds_load16s(min(at, static_cast<uint32_t>(i_last) << 8) + chunk, v ? vbase : kbase, dst);
        }
    };
    // V of a key that is masked for every row must not be multiplied: its weight is zero, but zero times a V that is not finite is NaN.
    // DUO: tiles behind the workgroup's last read V of the first tile instead (every row has it), and row block 0 leaves out the one
    // tile that only row block 1 has (64 rows of one head).
    const int second_only = DUO && p.hc == 1 ? (my_i0[0] + 31) / 32 + 1 : -1;
    const int li = lane & 15, dsel = (lane >> 4) & 1;
    const int k_row = (qi >> 2) * kGroupBytes + (qi & 3) * 256;
    const int k_off0 = k_row + 16 * ((hh + qi) & 3), k_off2 = k_row + 16 * ((hh + qi + 2) & 3);
    const int v_rho = (li >> 2) & 3;
    const int v_lane = kTileBytes + hh * kGroupBytes + v_rho * 256 + 32 * dsel + 8 * (li & 3);
    int v_off[4];
#pragma unroll
    for (int sgr = 0; sgr < 4; ++sgr) v_off[sgr] = v_lane + 64 * ((sgr + v_rho) & 3);
    typedef __attribute__((address_space(3))) bf16x4t* lds_ptr_t;
    auto read_k = [&](int slot, bf16x8 (&kf)[8]) __attribute__((always_inline)) {
        const unsigned char* kt = kvbuf + slot * kSlotBytes;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            kf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(kt + ((kk & 1) ? k_off2 : k_off0) + 64 * (kk >> 1)));
    };

    bf16x8 kf[2][8], vf[2][8], pb[2][2][2];
    f32x16 sc[2][2];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)kvbuf));

    // causal mask of tile t for row block rb (only the tiles on and past the diagonal need it)
    auto mask_tile = [&](f32x16& acc, int t, int rb) __attribute__((always_inline)) {
        const int dlt = my_i0[rb] - 32 * t;
        if (dlt >= 31 || !my_rows[rb]) return;               // (a row block that does not exist is not stored: no mask, and it holds up nobody)
        const uint64_t w = (dlt < -31 || t >= nblk) ? 0ull : ((kAll63 << (31 - dlt)) & kAll63);
        mask_elements<0>(acc, lane_keep_bits(w, w, 0u, 0u, qi + 4 - 4 * hh, 4 - 4 * hh), __float_as_uint(NEG_INF));
    };
    // One slot, written out in issue order: pieces are separated by scheduling barriers, so the matrix instructions
    // and the vector work alternate as listed.  MR: the row block whose matrix products are issued; VR = 1 - MR: the
    // row block whose softmax runs.  sq: stage whose scores are computed (HAS_Q); sq - 1: stage whose P V is
    // accumulated (HAS_P); sv: stage whose scores go through the softmax (HAS_S).
#define VS_FENCE() __builtin_amdgcn_sched_barrier(0)
    auto slot = [&](auto mr_tag, auto has_q, auto has_p, auto has_s, auto masked, auto spread, int sq, int sv) __attribute__((always_inline)) {
        constexpr int MR = decltype(mr_tag)::value, VR = 1 - MR;
        constexpr bool HAS_Q = decltype(has_q)::value, HAS_P = decltype(has_p)::value, HAS_S = decltype(has_s)::value;
        constexpr bool MASKED = decltype(masked)::value, SPREAD = decltype(spread)::value;
        auto qmfma = [&](int kk, int u) __attribute__((always_inline)) {
            if (kk == 0) {
                f32x16 zero;
#pragma unroll
                for (int e = 0; e < 16; ++e) zero[e] = 0.f;
                sc[MR][u] = mfma32(kf[u][0], qf[MR][0], zero);
            } else {
                sc[MR][u] = mfma32(kf[u][kk], qf[MR][kk], sc[MR][u]);
            }
        };
        const int left_out = second_only - 2 * pair_of(sq - 1);
        auto pmfma = [&](int idx) __attribute__((always_inline)) {
            const int u = idx >> 3, t = (idx >> 2) & 1, db = idx & 3;
            if (DUO && MASKED && MR == 0 && left_out == u) return;
            oacc[MR][db] = mfma32(vf[u][2 * db + t], pb[MR][u][t], oacc[MR][db]);
        };
        // vbase[sgr] / kbase_[par]: per-lane LDS addresses of the stage, everything else is an immediate offset
        auto vread = [&](int u, int j, const uint32_t (&vbase)[4]) __attribute__((always_inline)) {
            const uint32_t a0 = vbase[j >> 1] + u * kSlotBytes + 4 * (j & 1) * kGroupBytes;
            const bf16x4t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(a0));
            const bf16x4t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(a0 + 2 * kGroupBytes));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                vf[u][j][e] = lo[e];
                vf[u][j][4 + e] = hi[e];
            }
        };
        uint32_t vbase[4];                                   // V fragments of stage sq - 1
        if constexpr (MR == 0 && HAS_P) {
            const uint32_t sbase = DUO ? lds0 + wave * 2 * kSlotBytes : lds0 + 2 * ((sq + 2) % 3) * kSlotBytes;
#pragma unroll
            for (int sgr = 0; sgr < 4; ++sgr) {
                vbase[sgr] = sbase + v_off[sgr];
                asm volatile("" : "+v"(vbase[sgr]));
            }
        }
        // one V fragment of stage sq - 1 behind each of the 16 score products, in the order of use
        auto vread_share = [&](int j) __attribute__((always_inline)) { vread(j >> 3, 2 * (j & 3) + ((j >> 2) & 1), vbase); };
        auto kread = [&](int u, int kk, const uint32_t (&kb)[2]) __attribute__((always_inline)) {
            typedef const __attribute__((address_space(3))) uint4* lds_u4_t;
            kf[u][kk] = __builtin_bit_cast(bf16x8, *(lds_u4_t)(kb[kk & 1] + u * kSlotBytes + 64 * (kk >> 1)));
        };
        // DUO: what the wavefront requests for itself, a group of a tile behind each matrix instruction, as soon as the fragments that were in
        // the buffer are in registers, which is 46 matrix instructions before the first fragment of it is read:
        //   Y(sq - 1) 26 .. 31, X(sq) 0, 1   K of stage sq + 1, first tile      X(sq) 2 .. 9     K of stage sq + 1, second tile
        //   X(sq) 10 .. 17                   V of stage sq, first tile          X(sq) 18 .. 25   V of stage sq, second tile
        // (the waits count what has been requested since).  SPREAD: all these tiles exist, and are whole.
        const bool next = SPREAD || sq + 1 < nst, after_next = SPREAD || sq + 2 < nst;
        auto own_rows = [&](int st, int u) __attribute__((always_inline)) { return 32 * (2 * pair_of(st) + u); };
        auto own_piece = [&](auto matrix) __attribute__((always_inline)) {
            constexpr int JJ = decltype(matrix)::value;
            constexpr auto whole = std::bool_constant<SPREAD>{};
            if constexpr (DUO && HAS_Q && MR == 0) {
                if constexpr (JJ < 2) {
                    if (next) load_own(whole, 0, 0, std::integral_constant<int, JJ + 6>{}, own_rows(sq + 1, 0));
                } else if constexpr (JJ < 10) {
                    if constexpr (JJ == 2 && HAS_P) asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
                    if constexpr (JJ == 2 && !HAS_P) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    if (next) load_own(whole, 0, 1, std::integral_constant<int, JJ - 2>{}, own_rows(sq + 1, 1));
                } else if constexpr (JJ < 26) {
                    constexpr int U = JJ < 18 ? 0 : 1;
                    if constexpr (JJ == 10 && HAS_P) asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
                    if constexpr (JJ == 18) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    int row0 = own_rows(sq, U);
                    if constexpr (!SPREAD) row0 = row0 < 32 * nblk ? row0 : 0;
                    load_own(whole, 1, U, std::integral_constant<int, (JJ - 10) % 8>{}, row0);
                }
            }
            if constexpr (DUO && HAS_Q && MR == 1 && JJ >= 26) {
                if constexpr (JJ == 26) asm volatile("s_waitcnt lgkmcnt(2)" ::: "memory");
                if (after_next) load_own(whole, 0, 0, std::integral_constant<int, JJ - 26>{}, own_rows(sq + 2, 0));
            }
        };
        // V of stage sq - 1, first and second tile
        auto v_arrived = [&](int u) __attribute__((always_inline)) {
            if constexpr (DUO && MR == 0 && HAS_P) {
                if (HAS_Q && next) asm volatile("s_waitcnt vmcnt(14)" ::: "memory");
                else if (u == 0) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
                else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            }
        };
        v_arrived(0);
        if constexpr (!DUO && MR == 1) {
            // stage sq+1 has arrived (this wavefront's part; the barrier publishes all of it) and every wavefront
            // has left stage sq-1 behind: its buffer takes stage sq+2
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if (!SPREAD && sq + 2 < nst) load_stage(sq + 2);
            VS_FENCE();
        }
        // Softmax elements as a three-deep pipeline: step k scales element k, takes the exponential of element k-1 and adds
        // element k-2 to the row sum (packing a finished pair): no instruction uses the result of its predecessor.
        float mc = 0.f, lsum = 0.f;
        float tq[4] = {0.f, 0.f, 0.f, 0.f};                  // values in flight, indexed by element mod 4
        int estep = 0;
        auto pack_pair = [&](int u, int e, float x0, float x1) __attribute__((always_inline)) {   // weights of elements e - 1 and e
            const f32x2 two = {x0, x1};
            uint32_t packed = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
            asm volatile("" : "+v"(packed));
            const bf16x2 r = __builtin_bit_cast(bf16x2, packed);
            pb[VR][u][e >> 3][(e & 7) - 1] = r[0];
            pb[VR][u][e >> 3][e & 7] = r[1];
        };
        auto expstep = [&]() __attribute__((always_inline)) {
            if constexpr (HAS_S) {
                const int k = estep;
                if (k < 32) {
                    float t = fmaf(sc[VR][k >> 4][k & 15], p.c, -mc);
                    asm volatile("" : "+v"(t));
                    tq[k & 3] = t;
                }
                if (k >= 1 && k <= 32) {
                    float x = tq[(k - 1) & 3];
                    x = __builtin_amdgcn_exp2f(x);
                    asm volatile("" : "+v"(x));              // keeps the arithmetic at this place
                    tq[(k - 1) & 3] = x;
                }
                if (k >= 2 && k <= 33) {
                    const int idx = k - 2, u = idx >> 4, e = idx & 15;
                    lsum += tq[idx & 3];
                    asm volatile("" : "+v"(lsum));
                    if (e & 1) pack_pair(u, e, tq[(idx - 1) & 3], tq[idx & 3]);
                }
                ++estep;
            }
        };
        // 34 steps: over the first 31 matrix instructions (in front of the last is the look at the sum), or (MASKED) over the 26 behind the row maximum
        auto expsteps_upto = [&](int target) __attribute__((always_inline)) {
            while (estep < target) expstep();
        };
        auto exp_share = [&](int j) __attribute__((always_inline)) {   // behind matrix instruction j
            if constexpr (MASKED) expsteps_upto(((j - 5) * 34 + 25) / 26);
            else expsteps_upto(min(34, ((j + 1) * 34 + 30) / 31));
        };
        // ---- part 1: first matrix instructions | V fragments (X slot) | row maximum (MASKED) ----
        float mx0 = NEG_INF, mx1 = NEG_INF;
        float mxc[4];
        if constexpr (HAS_S && !MASKED) mc = m_run[VR] * p.c;
        if constexpr (HAS_S && MASKED) {
            mask_tile(sc[VR][0], 2 * pair_of(sv), VR);
            mask_tile(sc[VR][1], 2 * pair_of(sv) + 1, VR);
            VS_FENCE();
        }
        unroll<0, 6>([&](auto index) __attribute__((always_inline)) {
            constexpr int j = decltype(index)::value;
            if constexpr (HAS_Q) qmfma(j >> 1, j & 1);
            VS_FENCE();
            own_piece(index);
            if constexpr (MR == 0 && HAS_P) {
                vread_share(j);
            }
            if constexpr (!DUO && SPREAD && MR == 1 && (j & 1)) load_piece(sq + 2, j >> 1, true);
            if constexpr (HAS_S && !MASKED) exp_share(j);
            if constexpr (HAS_S && MASKED) {
                // row maximum: four independent chains (two per tile) of three-input maxima, one link of each per piece
                if (j < 4) {
#pragma unroll
                    for (int ch = 0; ch < 4; ++ch) {
                        const f32x16& a = sc[VR][ch >> 1];
                        const int b0 = 8 * (ch & 1);
                        if (j == 0) mxc[ch] = fmaxf(fmaxf(a[b0], a[b0 + 1]), a[b0 + 2]);
                        if (j == 1) mxc[ch] = fmaxf(fmaxf(mxc[ch], a[b0 + 3]), a[b0 + 4]);
                        if (j == 2) mxc[ch] = fmaxf(fmaxf(mxc[ch], a[b0 + 5]), a[b0 + 6]);
                        if (j == 3) mxc[ch] = fmaxf(mxc[ch], a[b0 + 7]);
                    }
                }
                if (j == 4) {
                    mx0 = fmaxf(mxc[0], mxc[1]);
                    mx1 = fmaxf(mxc[2], mxc[3]);
                }
            }
            VS_FENCE();
        });
        // mx: the lane's largest score of the stage; has the maximum moved?
        auto rescale = [&](float mx) __attribute__((always_inline)) -> bool {
            const float m_new = fmaxf(m_run[VR], half_swap_max(mx));
            if (!__ballot((m_new - m_run[VR]) * p.c > kRescaleThreshold)) return false;
            const float alpha = (m_new == NEG_INF) ? 1.f : __builtin_amdgcn_exp2f((m_run[VR] - m_new) * p.c);
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) oacc[VR][db][e] *= alpha;
            l_run[VR] *= alpha;
            m_run[VR] = m_new;
            return true;
        };
        if constexpr (HAS_S && MASKED) {
            rescale(fmaxf(mx0, mx1));
            mc = m_run[VR] == NEG_INF ? 0.f : m_run[VR] * p.c;
        }
        // the sum is complete: weigh the stage's scores anew if a row has grown
        auto look_again = [&]() __attribute__((always_inline)) {
            if (VS_MAY_HAVE_GROWN(lsum)) {                   // (P V of this stage and block is issued in the next slot)
                float mx[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    mx[u] = fmaxf(fmaxf(sc[VR][u][0], sc[VR][u][1]), sc[VR][u][2]);
#pragma unroll
                    for (int e = 3; e < 15; e += 2) mx[u] = fmaxf(fmaxf(mx[u], sc[VR][u][e]), sc[VR][u][e + 1]);
                    mx[u] = fmaxf(mx[u], sc[VR][u][15]);
                }
                if (rescale(fmaxf(mx[0], mx[1]))) {
                    mc = m_run[VR] * p.c;
                    lsum = 0.f;
#pragma unroll
                    for (int idx = 0; idx < 32; idx += 2) {
                        const int u = idx >> 4, e = idx & 15;
                        const float x0 = __builtin_amdgcn_exp2f(fmaf(sc[VR][u][e], p.c, -mc));
                        const float x1 = __builtin_amdgcn_exp2f(fmaf(sc[VR][u][e + 1], p.c, -mc));
                        lsum += x0;
                        lsum += x1;
                        pack_pair(u, e + 1, x0, x1);
                    }
                }
            }
        };
        // ---- part 2: remaining matrix instructions | K fragments (Y slot) | exponentials ----
        uint32_t kb[2];                                      // K fragments of stage sq + 1 (past the last stage: a stale slot, never used)
        if constexpr (MR == 1 && HAS_Q) {
            const uint32_t sbase = DUO ? lds0 + wave * 2 * kSlotBytes : lds0 + 2 * ((sq + 1) % 3) * kSlotBytes;
            kb[0] = sbase + k_off0;
            kb[1] = sbase + k_off2;
            asm volatile("" : "+v"(kb[0]), "+v"(kb[1]));
        }
        unroll<6, 16>([&](auto index) __attribute__((always_inline)) {   // 10 more score products
            constexpr int j = decltype(index)::value;
            if constexpr (HAS_Q) qmfma(j >> 1, j & 1);
            VS_FENCE();
            if constexpr (j == 8) v_arrived(1);
            own_piece(index);
            if constexpr (MR == 0 && HAS_P) vread_share(j);
            if constexpr (!DUO && SPREAD && MR == 1 && (j & 1)) load_piece(sq + 2, j >> 1, true);
            if constexpr (HAS_S) exp_share(j);
            VS_FENCE();
        });
        unroll<0, 16>([&](auto index) __attribute__((always_inline)) {   // 16 P V products
            constexpr int j = decltype(index)::value;
            if constexpr (HAS_S && !MASKED && j == 15) look_again();
            if constexpr (HAS_P) pmfma(j);
            VS_FENCE();
            if constexpr (DUO && MR == 1 && HAS_Q) {         // K of stage sq + 1, first and second tile
                if (j == 0 && next) asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
                if (j == 8 && next) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            }
            own_piece(std::integral_constant<int, 16 + j>{});
            if constexpr (MR == 1 && HAS_Q) {
                kread(j >> 3, j & 7, kb);
            }
            if constexpr (HAS_S) exp_share(16 + j);
            VS_FENCE();
        });
        if constexpr (HAS_S) {
            expsteps_upto(34);
            l_run[VR] += lsum;
        }
        VS_FENCE();
    };
#undef VS_FENCE

    using T = std::true_type;
    using F = std::false_type;
    using R0 = std::integral_constant<int, 0>;
    using R1 = std::integral_constant<int, 1>;
    // stages whose two tiles lie below the diagonal for both row blocks need no mask
    int nfree = min(my_i0[0], my_i0[1]) / 64;
    if constexpr (DUO) nfree = nfree > wave ? (nfree - wave - 1) / kWaves + 1 : 0;   // pairs wave, wave + 4, .. below nfree

    __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        m_run[rb] = NEG_INF;
        l_run[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[rb][db][e] = 0.f;
    }
    if constexpr (DUO) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
            unroll<0, 8>([&](auto grp) __attribute__((always_inline)) { load_own(std::false_type{}, 0, u, grp, 64 * wave + 32 * u); });
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
        load_stage(0);
        if (nst > 1) load_stage(1);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
    }
    read_k(DUO ? 2 * wave : 0, kf[0]);
    read_k(DUO ? 2 * wave + 1 : 1, kf[1]);
    if constexpr (DUO) {                                     // as Y(-1) would
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (nst > 1) unroll<0, 6>([&](auto grp) __attribute__((always_inline)) { load_own(std::false_type{}, 0, 0, grp, 64 * (kWaves + wave)); });
    }
    slot(R0{}, T{}, F{}, F{}, T{}, F{}, 0, 0);                // X(0): scores of block 0
    slot(R1{}, T{}, F{}, T{}, T{}, F{}, 0, 0);                // Y(0): scores of block 1; softmax of block 0
    if (nst > 1) {
        slot(R0{}, T{}, T{}, T{}, T{}, F{}, 1, 0);            // X(1): softmax of block 1 for stage 0
        // Y(i) and X(i + 1) have the softmax of stage i: from here on without a maximum, up to the diagonal
        const int to = __ballot(m_run[0] == NEG_INF || m_run[1] == NEG_INF) ? 0 : min(nst - 1, nfree);
        int i = 1;
        for (; i < to && (DUO ? i + 2 < to : i < nst - 3); ++i) {   // (stage i + 2 is loaded, and whole)
            slot(R1{}, T{}, T{}, T{}, F{}, T{}, i, i);
            slot(R0{}, T{}, T{}, T{}, F{}, T{}, i + 1, i);
        }
        for (; i < to; ++i) {
            slot(R1{}, T{}, T{}, T{}, F{}, F{}, i, i);
            slot(R0{}, T{}, T{}, T{}, F{}, F{}, i + 1, i);
        }
        for (; i < nst - 1; ++i) {
            slot(R1{}, T{}, T{}, T{}, T{}, F{}, i, i);
            slot(R0{}, T{}, T{}, T{}, T{}, F{}, i + 1, i);
        }
        slot(R1{}, T{}, T{}, T{}, T{}, F{}, nst - 1, nst - 1);
    }
    slot(R0{}, F{}, T{}, T{}, T{}, F{}, nst, nst - 1);        // X(nst): P V of block 0; softmax of block 1
    slot(R1{}, F{}, T{}, F{}, T{}, F{}, nst, nst);            // Y(nst): P V of block 1

    if constexpr (DUO) {
        __syncthreads();                                     // every buffer is idle
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) deposit_partial(smem, 2 * wave + rb, oacc[rb], m_run[rb], l_run[rb]);
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < 2; ++rb) finish_partials<kWaves>(p, smem, rb, 2, wave, my_head[rb], my_i0[rb]);
        return;
    }
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        const float l_tot = half_swap_sum(l_run[rb]);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        const int row = my_i0[rb] + qi;
        if (row < n_pos) {
            uint16_t* dst = p.o + (static_cast<size_t>(my_head[rb]) * p.nq + (row - p.pos0)) * kD;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f32x2 x01 = {oacc[rb][db][4 * a] * inv, oacc[rb][db][4 * a + 1] * inv};
                    const f32x2 x23 = {oacc[rb][db][4 * a + 2] * inv, oacc[rb][db][4 * a + 3] * inv};
                    const bf16x2 y01 = __builtin_convertvector(x01, bf16x2);
                    const bf16x2 y23 = __builtin_convertvector(x23, bf16x2);
                    uint2 out;
                    out.x = __builtin_bit_cast(uint32_t, y01);
                    out.y = __builtin_bit_cast(uint32_t, y23);
                    *reinterpret_cast<uint2*>(dst + 32 * db + 8 * a + 4 * hh) = out;
                }
            if (p.lse && hh == 0)
                p.lse[static_cast<size_t>(my_head[rb]) * p.nq + (row - p.pos0)] = l_tot > 0.f ? m_run[rb] * p.scale + __logf(l_tot) : NEG_INF;
        }
    }
}

template <bool DUO>
int launch_dense(AttnParams& p, hipStream_t stream) {
    static vs::PerDeviceOnce once;
    constexpr size_t lds = DUO ? kDuoBytes : kSmemBytes;
    const int rc_once = once.run(nullptr, [](int) -> int {
        VS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(&vs_dense_kernel<DUO>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   static_cast<int>(lds)));
        return VS_OK;
    });
    if (rc_once != VS_OK) return rc_once;
    p.kv_rows = p.n;
    p.n = p.pos0 + p.nq;
    const int BQ = (DUO ? 64 : 256) / p.hc;
    p.tiles = (p.nq + BQ - 1) / BQ;
    // one workgroup per (query tile, KV head, chunk of the group's heads), longest tiles first; workgroups are dealt
    // to the 8 XCDs round-robin, so KV head = block % kv_heads keeps a head's K / V in one XCD's L2
    const long long blocks = static_cast<long long>(p.kv_heads) * (p.group / p.hc) * p.tiles;
    if (blocks > 0x7fffffffLL) return VS_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(vs_dense_kernel<DUO>, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), lds, stream, p);
    VS_LAUNCH_CHECK();
    return VS_OK;
}

// More workgroups of the long form than that, but about one round of them or less: the call then takes as long as its longest workgroup,
// while the two-row-block form spreads the same work evenly, at a higher price per tile and per workgroup.  An estimate for the whole card
// (256 compute units at the 1.8 to 2 GHz that it holds under these kernels); a card cut into partitions would want other numbers.  Long form: 0.93 us per tile
// of the longest workgroup, or of the average over 256 compute units where that is more; DUO: 0.55 us per tile and row block of a SIMD and 7 us
// per round of workgroups.  That was before stages without a row maximum, from which the long form has gained more (it is now 0.53 to 0.62 us per tile,
// DUO 0.46), so the line leaves some time on the long form's side.  Here / there, us: 24 x 2048 (192 workgroups) 53 / 51, 8 / 2 x 6000 (188) 111 / 91,
// x 8192 (256) 159 / 145, 1 x 40000 (157) 666 / 388, x 65536 1180 / 972, 2 / 1 x 30000 534 / 427; not: 32 / 8 x 2048 (256) 49 / 59, x 3000 (375) 73 / 105,
// 8 / 2 x 16000 (500) 402 / 498, 2000 rows of 8192 (250) 197 / 233; on the wrong side: 16 x 4096 (256) 90 / 93, 8 / 2 x 10000 (314) 204 / 214, 32 / 8, 1500
// rows of 8192 (188) 167 / 181, of 32768 646 / 700, 1100 of 32768 (144) 559 / 623.
bool duo_is_faster(int q_heads, int64_t n_q, int64_t pos0) {
    const int64_t blocks = (n_q + 31) / 32, last = (pos0 + n_q + 31) / 32;
    const int64_t work = q_heads * (blocks * (last - blocks) + blocks * (blocks + 1) / 2);   // tiles x row blocks
    const int64_t rounds = (q_heads * blocks / 2 + 255) / 256;
    const int64_t average = work / (8 * 256);                // eight row blocks a workgroup
    return 0.55 * static_cast<double>(work) / 1024.0 + 7.0 * static_cast<double>(rounds) <
           0.95 * 0.93 * static_cast<double>(last > average ? last : average);
}

}  // namespace

extern "C" {

int vs_dense_prefill_chunk(const void* q, const void* k, const void* v, int q_heads, int kv_heads, int64_t n_q, int64_t n_kv,
                           int64_t pos0, float scale, void* o_bf16, float* lse, void* stream) {
    int rc = check_qkv(q, k, v, q_heads, kv_heads, n_kv, scale, o_bf16);
    if (rc != VS_OK) return rc;
    rc = check_chunk(n_q, n_kv, pos0);
    if (rc != VS_OK) return rc;
    AttnParams p{};
    p.q = static_cast<const uint16_t*>(q);
    p.k = static_cast<const uint16_t*>(k);
    p.v = static_cast<const uint16_t*>(v);
    p.o = static_cast<uint16_t*>(o_bf16);
    p.lse = lse;
    p.q_heads = q_heads;
    p.kv_heads = kv_heads;
    p.group = q_heads / kv_heads;
    p.index_per_q = 0;
    p.hc = heads_per_workgroup(p.group, false);
    p.n = static_cast<int>(n_kv);
    p.nq = static_cast<int>(n_q);
    p.pos0 = static_cast<int>(pos0);
    p.scale = scale;
    p.c = scale * 1.4426950408889634f;
    p.tile_counter = nullptr;
    // Workgroups for at most half of the compute units: split the keys of a row block over wavefronts instead.  At 128 workgroups,
    // vs_short_kernel there:
    // 128 heads x 200 15.8 us here, 14.5 there, 64 x 500 23.0 and 18.0, 32 x 1024 34.8 and 23.1, 32 / 8 x 1024 32.0 and 21.6,
    // 4 / 2 x 8192 187 and 94.  Beyond, long sequences still gain (152: 32 / 8 x 1200 35.9 and 30.7; 192: 24 x 2048 56.6 and 48.2),
    // short ones and long contexts lose (160: 160 x 200 16.5 and 20.0, 80 x 500 23.6 and 24.3; 152: 32 / 8, 1200 rows of 8192 keys
    // 191 and 211; 240: 64 / 16 x 900 33.8 and 37.5).
    // A wavefront that has one or two tiles in all stays here: one head (1, 8, 32 of them) x 64 6.0 to 6.3 us here, 6.7 to 6.9 there
    // (x 65 8.0 and 6.7), two heads of a group x 32 6.1 and 6.6 (x 64 7.2 and 6.7); four heads of a group x 32 7.3 and 6.8.
    const int64_t units = static_cast<int64_t>(kv_heads) * (p.group / p.hc) * ((n_q * p.hc + 255) / 256);
    const bool few_tiles = p.hc <= 2 && n_kv * p.hc <= 64;
    if (units <= kShortUnits && !few_tiles) {
        const int rows = vs::dense_lone(p.q_heads, p.nq, p.pos0) ? 1 : 2;
        p.hc = vs::short_heads(p.hc, rows);
        // Of these, more than 256 row blocks against at least 2048 keys: two row blocks per wavefront (DUO).  There / vs_short_kernel, us:
        // 8 x 2048 22 / 25, 16 / 4 x 2048 33 / 33, 12 x 2600 36 / 55, 8 / 2 x 2600 27 / 28, x 3800 40 / 44, 12 / 6 x 2600 35 / 36, 32 / 8, 500 rows of 2048 24 / 25,
        // 750 of 2100 38 / 39, 1024 of 4096 71 / 80, of 32768 530 / 636; with fewer keys the fill and the larger stages cost as much: 16 / 4 x 1700 29 / 26,
        // 24 x 1280 26 / 23, 32 / 8 x 1024 24 / 21.
        if (rows == 2 && n_kv >= kDuoKeys) return launch_dense<true>(p, static_cast<hipStream_t>(stream));
        return vs::launch_short_dense(p, rows, static_cast<hipStream_t>(stream));
    }
    if (n_kv >= kDuoKeys && duo_is_faster(q_heads, n_q, pos0)) {
        p.hc = vs::short_heads(p.hc, 2);
        return launch_dense<true>(p, static_cast<hipStream_t>(stream));
    }
    return launch_dense<false>(p, static_cast<hipStream_t>(stream));
}

int vs_dense_prefill(const void* q, const void* k, const void* v, int q_heads, int kv_heads, int64_t n, float scale,
                     void* o_bf16, float* lse, void* stream) {
    return vs_dense_prefill_chunk(q, k, v, q_heads, kv_heads, n, n, 0, scale, o_bf16, lse, stream);
}

}  // extern "C"
