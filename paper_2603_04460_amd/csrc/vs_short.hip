// Attention for launches with few row blocks (short sequences, short chunks of long ones, few heads), sparse and dense.
//
// The kernels of vs_attention.hip and vs_dense.hip give every row block of 32 query rows to one wavefront, which walks all
// its keys: a chunk of 500 rows is 64 workgroups on 256 compute units, each as long as the context.  Here a row block's
// tiles are dealt to several wavefronts; at the end their partial results (maximum, sum, O) meet in LDS and every wavefront
// finishes its share of the 128 channels.  A workgroup has 8 wavefronts, two per SIMD, one workgroup per compute unit.
// Arithmetic, tile layout, records and gather lists are those of vs_attention.hip.
//   vs_short_kernel  two row blocks (two query heads of the KV group, or 64 consecutive rows of one head) of four wavefronts, or four
//                    of two.  A stage is four 32-key tiles, wavefront (s, rb) takes tile s (and s + 2) of the stage for row block
//                    rb; two stages live in LDS.
//   vs_lone_kernel   one row block of eight wavefronts, each with LDS buffers of its own (vs::short_lone, at most 256 row blocks; dense up
//                    to 512, vs::dense_lone).
//
// Long dense calls with more row blocks than that go to the two-row-block form of vs_dense.hip.
//
// Measured (8 KV / 32 query heads unless stated): dense, 1024 x 1024 32 -> 22 us.  A step of vs_short_kernel (four tiles, 64 KB staged)
// takes 1.07 us while few workgroups run, 1.26 to 1.46 with one on every compute unit: the LDS (64 KB written, 128 KB of fragments
// read) and the chain barrier - fragment reads - scores - softmax - P V of a single tile per wavefront.
// Score products of a tile are one chain (a chain of matrix instructions runs as fast as two; two cost 16 adds).  Where it pays, tiles take the
// row maximum as it stands once every row has one (vs_attn_device.h): sparse with two or four row blocks (32 / 8 heads, 1000 rows of 40000
// keys 51.5 -> 49.3 us, 16384 rows of one head 102.5 -> 99.3; without 50.6 and 101.9), dense with one (8 / 2 heads, 1000 rows of 65536 keys
// 359 -> 335).  Dense with two row blocks has too few tiles per wavefront for it (32 / 8 heads x 900 20.0 us before, 19.5 now, 20.1 with it), and a
// sparse row block to itself is bound by its loads: 16 KB a tile at the 64 bytes a clock that a compute unit's vector memory takes, 256 clocks
// (n = 4096, below, 30.4 with it, 28.7 without).
// vs_lone_kernel: sparse, one head, n = 4096, 68 scattered columns and 190 offsets 51.7 -> 30.4 us with the preparation (111 in
// vs_attention.hip); dense, one head, 8192 x 8192 74 -> 45 us, 64 rows, 32 / 8 heads, against 32768 keys 280 -> 151 us.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "vs_attn_device.h"

namespace {

constexpr int kThreads = 512;
constexpr int kStage = 4;                      // tiles per stage
constexpr int kListCap = 256;                  // block list: kListCap / nsub entries per pass
constexpr int kGatherCap = 2432;               // gather list entries per pass
constexpr int kRecPad = 2 * kStage;            // dead records after the last listed block (a step looks one stage ahead)
constexpr size_t kRingBytes = 2 * kStage * kSlotBytes;
constexpr size_t kRecOff = kRingBytes;
constexpr size_t kGatherOff = kRecOff + (kListCap + 4 * kRecPad) * 16;
constexpr size_t kSparseLds = kGatherOff + kGatherCap * 4;
static_assert(kPartialBytes + 8 * 4 <= kRingBytes, "partial results in the idle ring");
static_assert(kSparseLds <= 160 * 1024, "one workgroup per compute unit");
static_assert(kGatherCap % (32 * kStage) == 0, "whole stages");

// Fragment addresses of a lane in an LDS slot, as in vs_attention.hip.
struct Fragments {
    int k_off0, k_off2, v_off[4];
    typedef __attribute__((address_space(3))) bf16x4t* lds_ptr_t;
    __device__ __forceinline__ explicit Fragments(int lane) {
        const int qi = lane & 31, hh = lane >> 5, li = lane & 15, dsel = (lane >> 4) & 1;
        const int k_row = (qi >> 2) * kGroupBytes + (qi & 3) * 256;
        k_off0 = k_row + 16 * ((hh + qi) & 3);
        k_off2 = k_row + 16 * ((hh + qi + 2) & 3);
        const int v_rho = (li >> 2) & 3;
        const int v_lane = kTileBytes + hh * kGroupBytes + v_rho * 256 + 32 * dsel + 8 * (li & 3);
#pragma unroll
        for (int sgr = 0; sgr < 4; ++sgr) v_off[sgr] = v_lane + 64 * ((sgr + v_rho) & 3);
    }
    __device__ __forceinline__ void read_k(const unsigned char* at, bf16x8 (&kf)[8]) const {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            kf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(at + ((kk & 1) ? k_off2 : k_off0) + 64 * (kk >> 1)));
    }
    // j = 2 db + t16: d block db, keys 16 t16 ..
    __device__ __forceinline__ void read_v(const unsigned char* at, int j, bf16x8& vf) const {
        const unsigned char* a0 = at + v_off[j >> 1] + 4 * (j & 1) * kGroupBytes;
        const bf16x4t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(a0));
        const bf16x4t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr_t)(a0 + 2 * kGroupBytes));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            vf[e] = lo[e];
            vf[4 + e] = hi[e];
        }
    }
};

// One wavefront's share of a row block: Q, the running maximum and sum, O.
struct RowBlock {
    bf16x8 qf[8];
    f32x16 oacc[4];
    float m_run, l_run;
    int settled;                                             // every row has a maximum, which moves only where a row has grown (vs_attn_device.h)

    // Q fragments: B operand of S^T = K Q^T; lane holds query qi, d = 16 kk + 8 hh .. +7
    __device__ __forceinline__ void init(const AttnParams& p, int head, int first, int qi, int hh) {
        const int row = min(first + qi, p.pos0 + p.nq - 1);  // rows that do not exist are not stored
        const uint16_t* src = p.q + (static_cast<size_t>(head) * p.nq + (row - p.pos0)) * kD + 8 * hh;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(src + 16 * kk));
        m_run = -INFINITY;
        l_run = 0.f;
        settled = 0;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[db][e] = 0.f;
    }
    // has the maximum moved?
    __device__ __forceinline__ bool new_maximum(const AttnParams& p, const f32x16& s) {
        float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
        for (int e = 3; e < 15; e += 2) mx = fmaxf(fmaxf(mx, s[e]), s[e + 1]);
        const float m_new = fmaxf(m_run, half_swap_max(fmaxf(mx, s[15])));
        if (!__ballot((m_new - m_run) * p.c > kRescaleThreshold)) return false;   // (false when both are -inf)
        const float alpha = (m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((m_run - m_new) * p.c);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[db][e] *= alpha;
        l_run *= alpha;
        m_run = m_new;
        return true;
    }
    // weights of a tile in bf16 and the lane's sum of them
    __device__ __forceinline__ float weigh(const AttnParams& p, const f32x16& s, bf16x8 (&pb)[2]) {
        const float mc = (m_run == -INFINITY) ? 0.f : m_run * p.c;
        float lsum[2] = {0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const float x0 = __builtin_amdgcn_exp2f(fmaf(s[e], p.c, -mc)), x1 = __builtin_amdgcn_exp2f(fmaf(s[e + 1], p.c, -mc));
            lsum[0] += x0;
            lsum[1] += x1;
            const f32x2 two = {x0, x1};
            const bf16x2 r = __builtin_convertvector(two, bf16x2);
            pb[e >> 3][e & 7] = r[0];
            pb[e >> 3][(e & 7) + 1] = r[1];
        }
        return lsum[0] + lsum[1];
    }
    // A tile: its K fragments are in registers, its V (v_there() waits for it) at `at`; kind: 0 nothing of it counts, 1 whole, 2 masked with the
    // keep-bits (bit 27 - 8a - c of element 4a + c) that keep() gives.  v_read(): the V fragments are in registers.
    // SETTLED: the maximum stays as it is, unless a row has grown
    template <bool SETTLED, class Keep, class Wait, class Load>
    __device__ __forceinline__ void tile(const AttnParams& p, const bf16x8 (&kf)[8], const Fragments& fr, const unsigned char* at, int kind,
                                         Keep keep, Wait v_there, Load v_read) {
        f32x16 s;
        bf16x8 vf[8], pb[2];
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) s = mfma32(kf[kk], qf[kk], s);
        __builtin_amdgcn_sched_barrier(0);
        v_there();
#pragma unroll
        for (int j = 0; j < 8; ++j) fr.read_v(at, j, vf[j]);
        __builtin_amdgcn_sched_barrier(0);
        if (kind == 2) mask_elements<0>(s, keep(), __float_as_uint(-INFINITY));
        if (kind) {
            if constexpr (!SETTLED) {
                new_maximum(p, s);
                settled = __builtin_amdgcn_readfirstlane(__ballot(m_run == -INFINITY) == 0ull ? 1 : 0);
            }
            float lsum = weigh(p, s, pb);
            if constexpr (SETTLED) {
                if (VS_MAY_HAVE_GROWN(lsum)) {
                    if (new_maximum(p, s)) lsum = weigh(p, s, pb);
                }
            }
            l_run += lsum;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        v_read();
        __builtin_amdgcn_sched_barrier(0);
        if (kind) {
#pragma unroll
            for (int t = 0; t < 2; ++t)                      // the four d blocks in turn: consecutive products are independent
#pragma unroll
                for (int db = 0; db < 4; ++db) oacc[db] = mfma32(vf[2 * db + t], pb[t], oacc[db]);
        }
    }
    // executed tiles of this wavefront in *tiles (null: none): their sum over the workgroup in thread 0 afterwards
    template <int SPLITS>
    __device__ __forceinline__ void merge(const AttnParams& p, unsigned char* smem, int first, int stride, int split, int head, int first_row,
                                          unsigned int* tiles) {
        unsigned int* const done = reinterpret_cast<unsigned int*>(smem + kPartialBytes);
        const int wave = first + stride * split;
        deposit_partial(smem, wave, oacc, m_run, l_run);
        if (tiles && (threadIdx.x & 63) == 0) done[wave] = *tiles;
        __syncthreads();
        if (tiles && threadIdx.x == 0)
            for (int w = 1; w < kThreads / 64; ++w) *tiles += done[w];
        finish_partials<SPLITS>(p, smem, first, stride, split, head, first_row);
    }
};

// keep-bits (bit 27 - 8a - c of element 4a + c) of a gathered tile: column <= row; cols: the tile's columns from 4 hh on
__device__ __forceinline__ uint32_t causal_columns(const int* cols, int row) {
    uint32_t keep = 0u;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int4 c4 = *reinterpret_cast<const int4*>(cols + 8 * a);
        keep |= (c4.x <= row ? 1u << (27 - 8 * a) : 0u) | (c4.y <= row ? 1u << (26 - 8 * a) : 0u) |
                (c4.z <= row ? 1u << (25 - 8 * a) : 0u) | (c4.w <= row ? 1u << (24 - 8 * a) : 0u);
    }
    return keep;
}

template <bool DENSE, int kRowBlocks>
__global__ __launch_bounds__(kThreads) void vs_short_kernel(const AttnParams p) {
    constexpr int kSplits = kThreads / 64 / kRowBlocks;      // wavefronts per row block
    static_assert(kStage % kSplits == 0, "whole steps");
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char* const kvbuf = smem;
    uint4* const list_rec = reinterpret_cast<uint4*>(smem + kRecOff);
    int* const glist = reinterpret_cast<int*>(smem + kGatherOff);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31, hh = lane >> 5;
    const int rb = wave % kRowBlocks, split = wave / kRowBlocks;
    const int rest = blockIdx.x / p.kv_heads, g = blockIdx.x % p.kv_heads;
    const int hchunks = p.group / p.hc;
    const int hchunk = rest % hchunks;
    const int tile = p.tiles - 1 - rest / hchunks;          // longest tiles first
    const int nsub = kRowBlocks / p.hc, BQ = 32 * nsub;
    const int i0 = p.pos0 + tile * BQ;                      // positions are absolute; the tile grid starts at the chunk
    const int n = p.n, n_pos = p.pos0 + p.nq;
    const int i_last = min(i0 + BQ, n_pos) - 1;
    const int my_head = g * p.group + hchunk * p.hc + rb % p.hc;
    const int my_sub = rb / p.hc;
    const int my_i0 = i0 + 32 * my_sub;
    const bool my_rows = my_i0 < n_pos;
    const uint16_t* __restrict__ kbase = p.k + static_cast<size_t>(g) * n * kD;
    const uint16_t* __restrict__ vbase = p.v + static_cast<size_t>(g) * n * kD;

    RowBlock row_block;
    row_block.init(p, my_head, my_i0, qi, hh);
    const Fragments fr(lane);
    // staging: wavefront w fills group w (rows 4 w + L / 16) of the K and of the V tile of every slot of the stage
    const int st_row = tid >> 4;
    const int st_rho = (lane >> 4) & 3;
    const uint32_t st_bk = static_cast<uint32_t>(16 * (4 * ((lane >> 2) & 3) + (((lane & 3) - st_rho) & 3)));
    const uint32_t st_bv = static_cast<uint32_t>(16 * (4 * ((((lane >> 2) & 3) - st_rho) & 3) + (lane & 3)));
    auto load_tile = [&](int row, int slot) __attribute__((always_inline)) {
        unsigned char* const dst = kvbuf + slot * kSlotBytes + wave * kGroupBytes;
        const uint32_t off = static_cast<uint32_t>(min(row, n_pos - 1)) << 8;  // rows behind the last position are masked, and not read
        lds_load16s(off + st_bk, kbase, dst);
        lds_load16s(off + st_bv, vbase, dst + kTileBytes);
    };
    // One tile for this wavefront: slot in LDS; need: mask with the keep-bits that keep() gives.
    auto compute = [&](auto settled, int slot, bool need, auto keep) __attribute__((always_inline)) {
        const unsigned char* const at = kvbuf + slot * kSlotBytes;
        bf16x8 kf[8];
        fr.read_k(at, kf);
        row_block.tile<decltype(settled)::value>(p, kf, fr, at, need ? 2 : 1, keep, [] {}, [] {});
    };
    // Pipeline over the stages of one phase: load(st, buf) requests the four tiles of stage st; step(t, slot) computes tile t, one of
    // this wavefront's.  One barrier per stage publishes stage st and frees the buffer of stage st - 1.
    auto run_phase = [&](int ntiles, auto load, auto step) __attribute__((always_inline)) {
        const int nst = (ntiles + kStage - 1) / kStage;
        load(0, 0);
        int st = 0;
        auto stage = [&](auto settled) __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): this wavefront's part of stage st has arrived
            __syncthreads();
            if (st + 1 < nst) load(st + 1, (st + 1) & 1);
#pragma unroll
            for (int u = split; u < kStage; u += kSplits) step(settled, kStage * st + u, kStage * (st & 1) + u);
            ++st;
        };
        if constexpr (DENSE) {                               // (never settled: the rule is at the top of this file)
            while (st < nst) stage(std::false_type{});
        } else {
            while (st < nst && !row_block.settled) stage(std::false_type{});
            while (st < nst) stage(std::true_type{});
        }
        __syncthreads();                                     // the ring and the lists are reused
    };
    unsigned int tiles_done = 0, staged_gather = 0, staged_block = 0;

    if constexpr (DENSE) {
        const int nblk = i_last / 32 + 1;
        run_phase(
            nblk,
            [&](int st, int buf) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < kStage; ++u) load_tile(32 * (kStage * st + u) + st_row, kStage * buf + u);
            },
            [&](auto settled, int t, int slot) __attribute__((always_inline)) {
                const int dlt = my_i0 - 32 * t;                               // offset of (row 0, key 0)
                if (dlt < -31 || !my_rows) return;
                compute(settled, slot, dlt < 31, [&]() __attribute__((always_inline)) {
                    const uint64_t w = (kAll63 << (31 - dlt)) & kAll63;       // offsets >= 0
                    return static_cast<uint32_t>(w >> (qi + 4 - 4 * hh));
                });
            });
    } else {
        const int ih = p.index_per_q ? my_head : g;
        const uint32_t* __restrict__ vbit = p.vbit + static_cast<size_t>(ih) * p.vw;
        const int32_t* __restrict__ iv = p.idx_v + static_cast<size_t>(ih) * p.cap_v;
        const int32_t* __restrict__ ncol = p.ncol32 + static_cast<size_t>(ih) * p.nq32;
        const int32_t* __restrict__ dl = p.dlist + static_cast<size_t>(ih) * p.dcap;
        const unsigned long long* __restrict__ wl = p.wlist + static_cast<size_t>(ih) * p.dcap * 4;
        const int qb0 = i0 >> 5;
        const int ndiag = p.ndiag[static_cast<size_t>(ih) * p.nq32 + qb0];
        const int ncand = ncol[i_last >> 5];
        int cursor = min(p.vfirst[ih], ncand);
        const int bcap = kListCap / nsub, rcap = bcap + kRecPad;
        const uint4* const my_rec = list_rec + my_sub * rcap;
        // 1. slash part: key blocks qb0 - delta in the order of the diagonal list, in rounds of bcap blocks
        for (int rbase = 0; rbase < ndiag; rbase += bcap) {
            const int count = min(bcap, ndiag - rbase);
            if (tid < count) {
                const int b = qb0 - dl[rbase + tid];
                const uint32_t xw = vbit[b];
                for (int r = 0; r < nsub; ++r)
                    list_rec[r * rcap + tid] = tile_record(p.gran, n_pos, i0 + 32 * r, b, wl[static_cast<size_t>(rbase + tid) * 4 + r], xw);
            } else if (tid < count + kRecPad) {
                for (int r = 0; r < nsub; ++r) list_rec[r * rcap + tid] = make_uint4(0u, 0u, 0u, 0u);
            }
            __syncthreads();
            staged_block += static_cast<unsigned int>(count);
            run_phase(
                count,
                [&](int st, int buf) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < kStage; ++u)
                        load_tile(32 * static_cast<int>(list_rec[kStage * st + u].w >> 2) + st_row, kStage * buf + u);
                },
                [&](auto settled, int t, int slot) __attribute__((always_inline)) {
                    const uint4* const rec = my_rec + t;
                    const uint32_t fl = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(rec->w));
                    if (!(fl & 1u)) return;
                    ++tiles_done;
                    compute(settled, slot, (fl & 2u) != 0u, [&]() __attribute__((always_inline)) {
                        const uint4 r = *rec;                // one broadcast read
                        const uint64_t wz = (static_cast<uint64_t>(r.y) << 32) | r.x;
                        return static_cast<uint32_t>(wz >> (qi + 4 - 4 * hh)) & (__builtin_bitreverse32(r.z) >> (4 - 4 * hh));
                    });
                });
        }
        // 2. vertical part: the causal columns, gathered row by row, in rounds of kGatherCap
        while (cursor < ncand) {
            const int count = min(ncand - cursor, kGatherCap);
            const int padded = (count + 32 * kStage - 1) / (32 * kStage) * (32 * kStage);
            for (int t = tid; t < padded; t += kThreads) glist[t] = t < count ? iv[cursor + t] : INT_MAX;
            const int last = last_column(iv + cursor, count, n_pos);
            cursor += count;
            __syncthreads();
            const int ntiles = (count + 31) >> 5;
            staged_gather += static_cast<unsigned int>(ntiles);
            run_phase(
                ntiles,
                [&](int st, int buf) __attribute__((always_inline)) {
#pragma unroll
                    for (int u = 0; u < kStage; ++u) load_tile(min(glist[32 * (kStage * st + u) + st_row], last), kStage * buf + u);
                },
                [&](auto settled, int t, int slot) __attribute__((always_inline)) {
                    const int* const cols = glist + 32 * t;
                    const int cmin = __builtin_amdgcn_readfirstlane(cols[0]), cmax = __builtin_amdgcn_readfirstlane(cols[31]);
                    if (!my_rows || cmin > my_i0 + 31) return;               // ascending, INT_MAX padding
                    ++tiles_done;
                    compute(settled, slot, cmax > my_i0, [&]() __attribute__((always_inline)) { return causal_columns(cols + 4 * hh, my_i0 + qi); });
                });
        }
    }

    // (the ring is idle: every phase ends with a barrier)
    row_block.merge<kSplits>(p, smem, rb, kRowBlocks, split, my_head, my_i0, DENSE ? nullptr : &tiles_done);
    if (!DENSE && tid == 0) add_statistics(p, tiles_done, staged_gather, staged_block);
}

// ---- one row block per workgroup ----
// Launches that do not even fill the chip with row blocks: every wavefront takes every eighth tile of the one row block, through a
// K and a V buffer of its own that it fills itself.  No barrier in the tile loop and no second buffer: the K buffer is refilled
// (tile t + 8) as soon as the K fragments of tile t are in registers, the V buffer likewise, so a load has the rest of the step to
// arrive, and a wavefront that waits leaves the SIMD to the other one.
constexpr int kLone = kThreads / 64;           // wavefronts = tiles in flight
constexpr size_t kLoneRing = kLone * kSlotBytes;
constexpr size_t kLoneRecOff = kLoneRing;
constexpr size_t kLoneGatherOff = kLoneRecOff + (kListCap + 1) * 16;
constexpr size_t kLoneLds = kLoneGatherOff + kGatherCap * 4;
static_assert(kPartialBytes + 8 * 4 <= kLoneRing, "partial results in the idle buffers");
static_assert(kLoneLds <= 160 * 1024, "one workgroup per compute unit");
static_assert(kGatherCap % 32 == 0, "whole tiles");

template <bool DENSE>
__global__ __launch_bounds__(kThreads) void vs_lone_kernel(const AttnParams p) {
    extern __shared__ __align__(16) unsigned char smem[];
    uint4* const list_rec = reinterpret_cast<uint4*>(smem + kLoneRecOff);
    int* const glist = reinterpret_cast<int*>(smem + kLoneGatherOff);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31, hh = lane >> 5;
    const int rest = blockIdx.x / p.kv_heads, g = blockIdx.x % p.kv_heads;
    const int my_head = g * p.group + rest % p.group;
    const int my_i0 = p.pos0 + 32 * (p.tiles - 1 - rest / p.group);          // longest row blocks first
    const int n = p.n, n_pos = p.pos0 + p.nq;
    const int i_last = min(my_i0 + 32, n_pos) - 1;
    const uint16_t* __restrict__ kbase = p.k + static_cast<size_t>(g) * n * kD;
    const uint16_t* __restrict__ vbase = p.v + static_cast<size_t>(g) * n * kD;
    unsigned char* const slot = smem + wave * kSlotBytes;

    RowBlock rb;
    rb.init(p, my_head, my_i0, qi, hh);
    const Fragments fr(lane);
    // staging: this wavefront fills all eight groups of its tile, lane L the piece of row 4 grp + L / 16
    const int st_rho = (lane >> 4) & 3;
    const uint32_t st_bk = static_cast<uint32_t>(16 * (4 * ((lane >> 2) & 3) + (((lane & 3) - st_rho) & 3)));
    const uint32_t st_bv = static_cast<uint32_t>(16 * (4 * ((((lane >> 2) & 3) - st_rho) & 3) + (lane & 3)));
    uint32_t off[8];                                         // byte offsets of the rows of the tile that is loaded next,
    int whole = -1;                                          // or its first row, if they all exist and stand one behind the other
    auto load = [&](uint32_t piece, const uint16_t* base, int offset) __attribute__((always_inline)) {   // into the own slot
        int w = wave;
        if constexpr (DENSE) asm volatile("" : "+s"(w));     // (the LDS addresses, merged over calls, ended up in vector registers)
        unsigned char* const dst = smem + w * kSlotBytes + offset;
        if (DENSE && whole >= 0) {
            lds_load_tile(static_cast<uint32_t>(st_rho) * 256u + piece, base + static_cast<size_t>(whole) * kD, dst);
            return;
        }
#pragma unroll
        for (int grp = 0; grp < 8; ++grp) lds_load16s(off[grp] + piece, base, dst + grp * kGroupBytes);
    };
    auto block_rows = [&](int b) __attribute__((always_inline)) {            // rows behind the last position are masked, and not read
        if constexpr (DENSE) {
            whole = 32 * b + 31 < n_pos ? 32 * b : -1;
            if (whole >= 0) return;
        }
#pragma unroll
        for (int grp = 0; grp < 8; ++grp) off[grp] = static_cast<uint32_t>(min(32 * b + 4 * grp + st_rho, n_pos - 1)) << 8;
    };
    // Tiles [0, ntiles) of a round, this wavefront's every eighth: rows(t) says what to load; need(t): 0 skip, 1 keep whole, 2 masked with
    // the keep-bits of keep(t)
    auto run = [&](int ntiles, auto rows, auto need, auto keep) __attribute__((always_inline)) {
        int t = wave;
        if (t >= ntiles) return;
        // (Q is waited for here: at its first use, in the tile loop, the compiler would wait for every load in flight, in every tile)
        __builtin_amdgcn_s_waitcnt(0x0F70);
        rows(t);
        load(st_bk, kbase, 0);
        load(st_bv, vbase, kTileBytes);
        auto step = [&](auto settled) __attribute__((always_inline)) {
            const bool more = t + kLone < ntiles;
            const int kind = need(t);
            if (more) rows(t + kLone);
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory"); // K of tile t (its V is younger)
            bf16x8 kf[8];
            fr.read_k(slot, kf);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (more) load(st_bk, kbase, 0);
            rb.tile<decltype(settled)::value>(
                p, kf, fr, slot, kind, [&]() __attribute__((always_inline)) { return keep(t); },
                [&]() __attribute__((always_inline)) {       // V of tile t (K of the next is younger)
                    if (more) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                },
                [&]() __attribute__((always_inline)) {
                    if (more) load(st_bv, vbase, kTileBytes);
                });
            t += kLone;
        };
        if constexpr (DENSE) {
            while (t < ntiles && !rb.settled) step(std::false_type{});
            while (t < ntiles) step(std::true_type{});
        } else {
            while (t < ntiles) step(std::false_type{});
        }
    };
    unsigned int tiles_done = 0, staged_gather = 0, staged_block = 0;
    if constexpr (DENSE) {
        auto dlt = [&](int t) { return my_i0 - 32 * t; };    // offset of (row 0, key 0)
        run(
            i_last / 32 + 1, block_rows, [&](int t) __attribute__((always_inline)) { return dlt(t) < -31 ? 0 : dlt(t) < 31 ? 2 : 1; },
            [&](int t) __attribute__((always_inline)) {
                const uint64_t w = (kAll63 << (31 - dlt(t))) & kAll63;       // offsets >= 0
                return static_cast<uint32_t>(w >> (qi + 4 - 4 * hh));
            });
    } else {
        const int ih = p.index_per_q ? my_head : g;
        const uint32_t* __restrict__ vbit = p.vbit + static_cast<size_t>(ih) * p.vw;
        const int32_t* __restrict__ iv = p.idx_v + static_cast<size_t>(ih) * p.cap_v;
        const int32_t* __restrict__ dl = p.dlist + static_cast<size_t>(ih) * p.dcap;
        const unsigned long long* __restrict__ wl = p.wlist + static_cast<size_t>(ih) * p.dcap * 4;
        const int qb0 = my_i0 >> 5;
        const int ndiag = p.ndiag[static_cast<size_t>(ih) * p.nq32 + qb0];
        const int ncand = p.ncol32[static_cast<size_t>(ih) * p.nq32 + (i_last >> 5)];
        int cursor = min(p.vfirst[ih], ncand);
        // rounds of up to kListCap listed blocks and kGatherCap columns; the gathered tiles follow the block tiles
        for (int rbase = 0; rbase < ndiag || cursor < ncand; rbase += kListCap) {
            const int nb = max(0, min(kListCap, ndiag - rbase)), count = min(ncand - cursor, kGatherCap);
            const int ng = (count + 31) >> 5;
            for (int t = tid; t < nb; t += kThreads) {
                const int b = qb0 - dl[rbase + t];
                list_rec[t] = tile_record(p.gran, n_pos, my_i0, b, wl[static_cast<size_t>(rbase + t) * 4], vbit[b]);
            }
            for (int t = tid; t < 32 * ng; t += kThreads) glist[t] = t < count ? iv[cursor + t] : INT_MAX;
            const int last = last_column(iv + cursor, count, n_pos);
            cursor += count;
            staged_block += static_cast<unsigned int>(nb);
            staged_gather += static_cast<unsigned int>(ng);
            __syncthreads();
            run(
                nb + ng,
                [&](int t) __attribute__((always_inline)) {
                    if (t < nb) {
                        block_rows(static_cast<int>(__builtin_amdgcn_readfirstlane(list_rec[t].w) >> 2));
                    } else {
#pragma unroll
                        for (int grp = 0; grp < 8; ++grp)
                            off[grp] = static_cast<uint32_t>(min(glist[32 * (t - nb) + 4 * grp + st_rho], last)) << 8;
                    }
                },
                [&](int t) __attribute__((always_inline)) {
                    int kind;
                    if (t < nb) {
                        const uint32_t fl = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(list_rec[t].w));
                        kind = fl & 1u ? ((fl & 2u) ? 2 : 1) : 0;
                    } else {
                        // ascending, INT_MAX padding; columns behind the row block are listed where a chunk starts inside a key block
                        const int* const cols = glist + 32 * (t - nb);
                        const int cmin = __builtin_amdgcn_readfirstlane(cols[0]), cmax = __builtin_amdgcn_readfirstlane(cols[31]);
                        kind = cmin > my_i0 + 31 ? 0 : cmax > my_i0 ? 2 : 1;
                    }
                    tiles_done += kind ? 1u : 0u;
                    return kind;
                },
                [&](int t) __attribute__((always_inline)) {
                    if (t < nb) {
                        const uint4 r = list_rec[t];         // one broadcast read
                        const uint64_t wz = (static_cast<uint64_t>(r.y) << 32) | r.x;
                        return static_cast<uint32_t>(wz >> (qi + 4 - 4 * hh)) & (__builtin_bitreverse32(r.z) >> (4 - 4 * hh));
                    }
                    return causal_columns(glist + 32 * (t - nb) + 4 * hh, my_i0 + qi);
                });
            __syncthreads();                                 // the lists are reused
        }
    }
    __syncthreads();                                         // every buffer is idle: the partial results take their place
    rb.merge<kLone>(p, smem, 0, 1, wave, my_head, my_i0, DENSE ? nullptr : &tiles_done);
    if (!DENSE && tid == 0) add_statistics(p, tiles_done, staged_gather, staged_block);
}

template <bool DENSE, int ROWS>
int launch_short(AttnParams& p, hipStream_t stream) {
    constexpr size_t lds = ROWS == 1 ? (DENSE ? kLoneRing : kLoneLds) : (DENSE ? kRingBytes : kSparseLds);
    void (*kernel)(AttnParams);
    if constexpr (ROWS == 1) kernel = &vs_lone_kernel<DENSE>;
    else kernel = &vs_short_kernel<DENSE, ROWS>;
    static vs::PerDeviceOnce once;
    const int rc = once.run(nullptr, [kernel](int) -> int {
        VS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
        return VS_OK;
    });
    if (rc != VS_OK) return rc;
    const int BQ = 32 * (ROWS / p.hc);
    p.tiles = (p.nq + BQ - 1) / BQ;
    // KV head = block % kv_heads: workgroups are dealt to the 8 XCDs round-robin, so a head's K / V stay in one XCD's L2
    const long long blocks = static_cast<long long>(p.kv_heads) * (p.group / p.hc) * p.tiles;
    if (blocks > 0x7fffffffLL) return VS_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), lds, stream, p);
    VS_LAUNCH_CHECK();
    return VS_OK;
}

}  // namespace

namespace vs {
int launch_short_dense(AttnParams& p, int rows, hipStream_t stream) {
    return rows == 1 ? launch_short<true, 1>(p, stream) : launch_short<true, 2>(p, stream);
}
int launch_short_sparse(AttnParams& p, int rows, hipStream_t stream) {
    return rows == 1 ? launch_short<false, 1>(p, stream) : rows == 2 ? launch_short<false, 2>(p, stream) : launch_short<false, 4>(p, stream);
}
}  // namespace vs
