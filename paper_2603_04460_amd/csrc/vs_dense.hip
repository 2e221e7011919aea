// Dense causal attention for gfx950 on the layout of the sparse kernel (bf16 Q / K / V, head dimension 128, GQA).
//
// Four wavefronts per workgroup, one per SIMD, each owning TWO 32-row blocks of the workgroup's 8 (hc query heads of
// the KV group times 8 / hc consecutive 32-row sub-blocks).  Every K / V fragment read from LDS feeds two matrix
// instructions, one per row block, which halves the LDS reads per flop against one row block per wavefront.  The
// arithmetic per row block (S^T = K Q^T, joint softmax over a stage of two 32-key tiles with a lazily updated
// maximum, O^T = V^T P^T) and the LDS tile layout are those of the sparse kernel.
//
// A SIMD issues about one vector instruction per 4-5 clocks whichever wavefront it comes from (an exponential
// takes 16), while a 32x32x16 matrix instruction occupies the matrix core for 32: the softmax of a stage costs
// more issue time than its matrix products cost matrix time, so the kernel is bound by the instruction stream
// and is written to keep that stream short and free of waits.  With one wavefront per SIMD the overlap of the
// softmax with the matrix core comes from inside the wavefront: the two row blocks run half a stage apart and
// each slot is written out in issue order, matrix and vector instructions alternating.
//   slot X(i): matrix: scores of block 0 for stage i, then P V of block 0 for stage i-1;  vector: softmax of block 1, stage i-1
//   slot Y(i): matrix: scores of block 1 for stage i, then P V of block 1 for stage i-1;  vector: softmax of block 0, stage i
// V fragments of stage i-1 are read at the start of X(i), K fragments of stage i+1 in Y(i) after the scores of
// block 1; one barrier per stage, in Y(i), publishes stage i+1 and frees the buffer of stage i-1 for stage i+2.
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
constexpr int kShortUnits = 128;               // workgroups up to which the keys of a row block are split
constexpr int kDuoKeys = 2048;

// DUO: few row blocks.  The workgroup has two row blocks, and every wavefront owns both; the keys are split over the wavefronts, which
// take stages of two tiles in turn, each through a K and a V buffer of its own that it fills itself (no barrier): stage i of
// wavefront w are the tiles 2 (4 i + w) and the next.  The K fragments of a stage are read in the Y slot before it, its V fragments in the X slot
// after it, so K of the next stage is requested in the X slot and V of this one in the Y slot, between the matrix instructions, and
// has a slot or more to arrive.  Against vs_short_kernel (one row block per wavefront, tiles shared by two wavefronts), which is bound by the
// LDS (64 KB staged and 128 KB of fragments read for four tiles, loads alone 221 us of 322), half the fragments are read: 500 rows
// against 32768 keys, 32 / 8 heads, 322 -> 282 us (another box 361 -> 289), 300 rows 282 -> 214, one head of 16384 143 -> 111.
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
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) {
        m_run[rb] = NEG_INF;
        l_run[rb] = 0.f;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[rb][db][e] = 0.f;
    }

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
    auto load_stage = [&](int st) __attribute__((always_inline)) {
        const int buf = st % 3;
        if (2 * st + 1 < nblk && 64 * st + 63 < n) {
            // every row of the stage exists: uniform base + per-thread offset, no address arithmetic per load
            const uint16_t* ks = kbase + static_cast<size_t>(64 * st) * kD;
            const uint16_t* vs_ = vbase + static_cast<size_t>(64 * st) * kD;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    unsigned char* dst = kvbuf + (2 * buf + u) * kSlotBytes + (wave + 4 * h) * kGroupBytes;
                    lds_load16s(voff_k[u][h], ks, dst);
                    lds_load16s(voff_v[u][h], vs_, dst + kTileBytes);
                }
            return;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int t = 2 * st + u;
                int row = 32 * t + st_row + 16 * h;
                if (t >= nblk || row >= n) row = 0;          // masked anyway: no predicate on the load (every row has key 0)
                unsigned char* dst = kvbuf + (2 * buf + u) * kSlotBytes + (wave + 4 * h) * kGroupBytes;
                const size_t off = static_cast<size_t>(row) * kD;
                lds_load16(kbase + off + st_ck * 8, dst);
                lds_load16(vbase + off + st_cv * 8, dst + kTileBytes);
            }
    };
    // DUO: one group of four rows of the wavefront's own tiles, row (lane / 16) of it; row0: first rows of the tiles; piece: 0 .. 15 of
    // K, then of V.  Rows behind the workgroup's last are masked and read that one.
    unsigned char* const own = kvbuf + wave * 2 * kSlotBytes;
    auto load_own = [&](int row0_0, int row0_1, int piece) __attribute__((always_inline)) {
        const int v = piece >> 4, u = (piece >> 3) & 1, grp = piece & 7;
        const uint32_t chunk = static_cast<uint32_t>(v ? st_cv : st_ck) * 16u;
        const uint32_t at = static_cast<uint32_t>((u ? row0_1 : row0_0) + 4 * grp + st_rho) * 256u;
        lds_load16s(min(at, static_cast<uint32_t>(i_last) << 8) + chunk, v ? vbase : kbase, own + u * kSlotBytes + v * kTileBytes + grp * kGroupBytes);
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
        if (dlt >= 31 && my_rows[rb]) return;
        const uint64_t w = (dlt < -31 || !my_rows[rb] || t >= nblk) ? 0ull : (dlt >= 31 ? kAll63 : ((kAll63 << (31 - dlt)) & kAll63));
        mask_elements<0>(acc, lane_keep_bits(w, w, 0u, 0u, qi + 4 - 4 * hh, 4 - 4 * hh), __float_as_uint(NEG_INF));
    };
    // One slot, written out in issue order: pieces are separated by scheduling barriers, so the matrix instructions
    // and the vector work alternate as listed.  MR: the row block whose matrix products are issued; VR = 1 - MR: the
    // row block whose softmax runs.  sq: stage whose scores are computed (HAS_Q); sq - 1: stage whose P V is
    // accumulated (HAS_P); sv: stage whose scores go through the softmax (HAS_S).
#define VS_FENCE() __builtin_amdgcn_sched_barrier(0)
    auto slot = [&](auto mr_tag, auto has_q, auto has_p, auto has_s, auto masked, int sq, int sv) __attribute__((always_inline)) {
        constexpr int MR = decltype(mr_tag)::value, VR = 1 - MR;
        constexpr bool HAS_Q = decltype(has_q)::value, HAS_P = decltype(has_p)::value, HAS_S = decltype(has_s)::value;
        constexpr bool MASKED = decltype(masked)::value;
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
        auto kread = [&](int u, int kk, const uint32_t (&kb)[2]) __attribute__((always_inline)) {
            typedef const __attribute__((address_space(3))) uint4* lds_u4_t;
            kf[u][kk] = __builtin_bit_cast(bf16x8, *(lds_u4_t)(kb[kk & 1] + u * kSlotBytes + 64 * (kk >> 1)));
        };
        if constexpr (DUO && MR == 0 && HAS_P) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // V of stage sq - 1
        if constexpr (!DUO && MR == 1) {
            // stage sq+1 has arrived (this wavefront's part; the barrier publishes all of it) and every wavefront
            // has left stage sq-1 behind: its buffer takes stage sq+2
            __builtin_amdgcn_s_waitcnt(0x0F70);
            __syncthreads();
            if (sq + 2 < nst) load_stage(sq + 2);
            VS_FENCE();
        }
        // ---- part 1: first matrix instructions | V fragments (X slot) | row maximum ----
        float mx0 = NEG_INF, mx1 = NEG_INF;
        float mxc[4];
        if constexpr (HAS_S && MASKED) {
            mask_tile(sc[VR][0], 2 * pair_of(sv), VR);
            mask_tile(sc[VR][1], 2 * pair_of(sv) + 1, VR);
            VS_FENCE();
        }
        uint32_t vbase[4];                                   // V fragments of stage sq - 1
        if constexpr (MR == 0 && HAS_P) {
            const uint32_t sbase = DUO ? lds0 + wave * 2 * kSlotBytes : lds0 + 2 * ((sq + 2) % 3) * kSlotBytes;
#pragma unroll
            for (int sgr = 0; sgr < 4; ++sgr) {
                vbase[sgr] = sbase + v_off[sgr];
                asm volatile("" : "+v"(vbase[sgr]));
            }
        }
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            if constexpr (HAS_Q) qmfma(j >> 1, j & 1);
            VS_FENCE();
            if constexpr (MR == 0 && HAS_P) {
                // V fragments of stage sq-1: 16 fragments over 6 pieces
#pragma unroll
                for (int f = 3 * j; f < min(3 * j + 3, 16); ++f) vread(f >> 3, f & 7, vbase);
            }
            if constexpr (HAS_S) {
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
        }
        if constexpr (HAS_S) {
            const float m_new = fmaxf(m_run[VR], half_swap_max(fmaxf(mx0, mx1)));
            if (__ballot((m_new - m_run[VR]) * p.c > kRescaleThreshold)) {
                const float alpha = (m_new == NEG_INF) ? 1.f : __builtin_amdgcn_exp2f((m_run[VR] - m_new) * p.c);
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[VR][db][e] *= alpha;
                l_run[VR] *= alpha;
                m_run[VR] = m_new;
            }
        }
        // ---- part 2: remaining matrix instructions | K fragments (Y slot) | exponentials ----
        const float mc = (!HAS_S || m_run[VR] == NEG_INF) ? 0.f : m_run[VR] * p.c;
        float lsum = 0.f;
        // Softmax elements as a three-deep pipeline: step k scales element k, takes the exponential of element k-1 and adds
        // element k-2 to the row sum (packing a finished pair): no instruction uses the result of its predecessor.
        float tq[3] = {0.f, 0.f, 0.f};                       // values in flight, indexed by element mod 3
        int estep = 0;
        auto expstep = [&]() __attribute__((always_inline)) {
            if constexpr (HAS_S) {
                const int k = estep;
                if (k < 32) {
                    float t = fmaf(sc[VR][k >> 4][k & 15], p.c, -mc);
                    asm volatile("" : "+v"(t));
                    tq[k % 3] = t;
                }
                if (k >= 1 && k <= 32) {
                    float x = tq[(k - 1) % 3];
                    x = __builtin_amdgcn_exp2f(x);
                    asm volatile("" : "+v"(x));              // keeps the arithmetic at this place
                    tq[(k - 1) % 3] = x;
                }
                if (k >= 2 && k <= 33) {
                    const int idx = k - 2, u = idx >> 4, e = idx & 15;
                    const float x = tq[idx % 3];
                    lsum += x;
                    asm volatile("" : "+v"(lsum));
                    sc[VR][u][e] = x;
                    if (e & 1) {
                        const f32x2 two = {sc[VR][u][e - 1], sc[VR][u][e]};
                        const bf16x2 r = __builtin_convertvector(two, bf16x2);
                        uint32_t packed = __builtin_bit_cast(uint32_t, r);
                        asm volatile("" : "+v"(packed));
                        const bf16x2 r2 = __builtin_bit_cast(bf16x2, packed);
                        pb[VR][u][e >> 3][(e & 7) - 1] = r2[0];
                        pb[VR][u][e >> 3][e & 7] = r2[1];
                    }
                }
                ++estep;
            }
        };
        // 34 steps over the 26 matrix instructions of this part
        auto expsteps_upto = [&](int target) __attribute__((always_inline)) {
            while (estep < target) expstep();
        };
        uint32_t kb[2];                                      // K fragments of stage sq + 1 (past the last stage: a stale slot, never used)
        if constexpr (MR == 1 && HAS_Q) {
            const uint32_t sbase = DUO ? lds0 + wave * 2 * kSlotBytes : lds0 + 2 * ((sq + 1) % 3) * kSlotBytes;
            kb[0] = sbase + k_off0;
            kb[1] = sbase + k_off2;
            asm volatile("" : "+v"(kb[0]), "+v"(kb[1]));
        }
        // DUO: K of stage sq + 1 is requested in the X slot, V of stage sq in the Y slot; the fragments that were read from these buffers
        // are in registers
        constexpr bool LOADS = DUO && HAS_Q;
        const bool next = sq + 1 < nst;
        if constexpr (LOADS && MR == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int load_pair = pair_of(MR == 0 ? sq + 1 : sq);
        int row0[2] = {64 * load_pair, 64 * load_pair + 32};
        if constexpr (MASKED && MR == 1) {                   // (without a mask every tile is the workgroup's)
            row0[0] = 2 * load_pair < nblk ? row0[0] : 0;
            row0[1] = 2 * load_pair + 1 < nblk ? row0[1] : 0;
        }
        auto loads_upto = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
            for (int piece = 0; piece < 32; ++piece)
                if (piece >= from && piece < to && (piece >= 16 || next)) load_own(row0[0], row0[1], piece);
        };
#pragma unroll
        for (int j = 6; j < 16; ++j) {                       // 10 more score products
            if constexpr (HAS_Q) qmfma(j >> 1, j & 1);
            VS_FENCE();
            if constexpr (LOADS && MR == 0) loads_upto((j - 6) * 16 / 26, (j - 5) * 16 / 26);
            if constexpr (LOADS && MR == 1) loads_upto(16 + (j - 6) * 16 / 10, 16 + (j - 5) * 16 / 10);
            if constexpr (HAS_S) expsteps_upto(((j - 6 + 1) * 34 + 25) / 26);
            VS_FENCE();
        }
        if constexpr (DUO && MR == 1 && HAS_Q) {             // K of stage sq + 1 (V of stage sq is younger)
            if (next) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {                       // 16 P V products
            if constexpr (HAS_P) pmfma(j);
            VS_FENCE();
            if constexpr (LOADS && MR == 0) loads_upto((10 + j) * 16 / 26, (11 + j) * 16 / 26);
            if constexpr (MR == 1 && HAS_Q) {
                kread(j >> 3, j & 7, kb);
            }
            if constexpr (HAS_S) expsteps_upto(((10 + j + 1) * 34 + 25) / 26);
            VS_FENCE();
        }
        if constexpr (HAS_S) {
            expsteps_upto(34);
            l_run[VR] += lsum;
        }
        VS_FENCE();
    };
#undef VS_FENCE

    __builtin_amdgcn_s_waitcnt(0x0F70);
    if constexpr (DUO) {
#pragma unroll
        for (int piece = 0; piece < 16; ++piece) load_own(64 * wave, 64 * wave + 32, piece);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    } else {
        load_stage(0);
        if (nst > 1) load_stage(1);
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
    }
    read_k(DUO ? 2 * wave : 0, kf[0]);
    read_k(DUO ? 2 * wave + 1 : 1, kf[1]);
    using T = std::true_type;
    using F = std::false_type;
    using R0 = std::integral_constant<int, 0>;
    using R1 = std::integral_constant<int, 1>;
    // stages whose two tiles lie below the diagonal for both row blocks need no mask
    int nfree = (my_rows[0] && my_rows[1]) ? min(my_i0[0], my_i0[1]) / 64 : 0;
    if constexpr (DUO) nfree = nfree > wave ? (nfree - wave - 1) / kWaves + 1 : 0;   // pairs wave, wave + 4, .. below nfree
    slot(R0{}, T{}, F{}, F{}, T{}, 0, 0);                    // X(0): scores of block 0
    slot(R1{}, T{}, F{}, T{}, T{}, 0, 0);                    // Y(0): scores of block 1; softmax of block 0
    int i = 1;
    for (; i < min(nst, nfree); ++i) {
        slot(R0{}, T{}, T{}, T{}, F{}, i, i - 1);
        slot(R1{}, T{}, T{}, T{}, F{}, i, i);
    }
    for (; i < nst; ++i) {
        slot(R0{}, T{}, T{}, T{}, T{}, i, i - 1);
        slot(R1{}, T{}, T{}, T{}, T{}, i, i);
    }
    slot(R0{}, F{}, T{}, T{}, T{}, nst, nst - 1);            // X(nst): P V of block 0; softmax of block 1
    slot(R1{}, F{}, T{}, F{}, T{}, nst, nst);                // Y(nst): P V of block 1

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
// per round of workgroups.  Here / there, us: 24 x 2048 (192 workgroups) 57 / 46, 16 x 4096 (256) 103 / 91, 8 / 2 x 6000 (188) 139 / 95, x 8192 (256)
// 191 / 154, x 10000 (314) 301 / 232, 1 x 40000 (157) 1134 / 439, 32 / 8, 1500 rows of 8192 (188) 237 / 196, of 32768 927 / 776, 1100 of 32768
// (144) 926 / 720; not: 32 / 8 x 2048 (256) 60 / 66, x 3000 (375) 84 / 108, 8 / 2 x 16000 (500) 448 / 543, 2048 rows of 8192 (256) 221 / 252.
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
        const int rows = vs::short_lone(p.q_heads, p.nq) ? 1 : 2;
        p.hc = vs::short_heads(p.hc, rows);
        // Of these, more than 256 row blocks against at least 2048 keys: two row blocks per wavefront (DUO).  There / vs_short_kernel, us:
        // 8 x 2048 22 / 25, 16 / 4 x 2048 33 / 33, 12 x 2600 79 / 80, 32 / 8, 500 rows of 2048 24 / 26, 1024 of 4096 73 / 80, of 32768 567 / 648;
        // with fewer keys the fill and the larger stages cost as much: 16 / 4 x 1700 27 / 26, 24 x 1280 25 / 24, 32 / 8 x 1024 24 / 22,
        // 128 x 200 18 / 15 (but 8 / 2 x 1500 17 / 19).
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
