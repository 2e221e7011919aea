// Distillation step of the VSIndexer (Sec. "Vertical-Slash Aggregation for Distillation Training", paragraph "Loss
// function design"): loss L = KL(A^_v || A_v) + KL(A^_s || A_s) between the indexer's two score vectors and the
// aggregated attention of the frozen model (vs_aggregate's outputs), and the gradient of L with respect to the
// indexer's parameters W_U, b_U, W_V, W_S.  The optimizer is the caller's.
//
//   1. forward: the inference kernels (vs_index_score) give A^_v, A^_s;
//   2. per (head, direction): KL = sum_t A^_t (ln A^_t - ln max(A_t, eps)) and the gradient with respect to the logits,
//      g_t = A^_t ((ln A^_t - ln A_t) - KL) / heads  (fp64 sums over blocks of 1024 tokens, added in a fixed order);
//   3. backward through the two-layer net with the hidden activations recomputed on the matrix cores.  Here the
//      up-projection runs as U = X W_U (tokens on the M axis, hidden units on the N axis), so that a lane holds 16 TOKENS
//      of ONE hidden unit: the token sums dW_V[u] = sum_t g_v z_u, dW_S, db_U are in-lane, and the pre-activation
//      gradients, rounded to two bf16 terms, are already the B operand of the second contraction
//      dW_U^T[c, u] = sum_t X[t, c] dpre[t, u], whose A operand X^T comes from LDS through the transposing read.
//      Every workgroup owns 128 hidden units (one 32-unit slice per wavefront, W_U fragments and the dW_U^T sums resident
//      in registers: one wavefront per SIMD) and a strided set of 32-token blocks.  Its partial sums, in fp32 over at most
//      1/256 of the blocks (or eight) whatever the width, go to the workspace and a last kernel adds them up in fp64, in a
//      fixed order (no float atomics: the step is deterministic).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "vs_common.h"
#include "vs_wave.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4t __attribute__((__vector_size__(4 * sizeof(__bf16))));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kThreads = 256;
constexpr int kUnitsPerWg = 128;               // 4 wavefronts x 32 hidden units
constexpr int kTokTile = 32;
constexpr int kXPitch = 512;                   // bytes per token row of the X tile in LDS (K then V, bf16)
constexpr int kXTile = kTokTile * kXPitch;
constexpr int kXBufs = 4;                      // tiles of blocks i - 1 (dW_U), i, i + 1 (U) and i + 2 (in flight)
constexpr int kPartials = 256;                 // an fp32 partial sum is over at most 1 / kPartials of the blocks,
constexpr int kPartBlocks = 8;                 // or over this many where that is more
constexpr int kKlThreads = 256;
constexpr int kKlBlock = 1024;                 // tokens per partial KL sum

__device__ __forceinline__ double block_sum(double x, double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
    __syncthreads();
    if (lane == 0) red[wave] = x;
    __syncthreads();
    double s = 0.0;
    for (int w = 0; w < kKlThreads / 64; ++w) s += red[w];
    return s;
}

// KL sums of 1024 tokens of one (head, direction) per workgroup.  (One workgroup per (head, direction) took 95 us at 8 x
// 32768 tokens: the two fp64 logarithms per token need the whole chip, not 16 compute units; this kernel and the next take
// 6.4 us each.)
__global__ __launch_bounds__(kKlThreads) void train_kl_kernel(const float* __restrict__ p_v, const float* __restrict__ p_s,
                                                               const float* __restrict__ t_v, const float* __restrict__ t_s, int n,
                                                               float eps, double* __restrict__ kl) {
    __shared__ double red[kKlThreads / 64];
    const int h = blockIdx.y, dir = blockIdx.z;
    const float* __restrict__ p = (dir == 0 ? p_v : p_s) + static_cast<size_t>(h) * n;
    const float* __restrict__ q = (dir == 0 ? t_v : t_s) + static_cast<size_t>(h) * n;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < kKlBlock / kKlThreads; ++i) {
        const int t = blockIdx.x * kKlBlock + i * kKlThreads + threadIdx.x;
        if (t < n) {
            const float pt = p[t];
            if (pt > 0.f) acc += static_cast<double>(pt) * (log(static_cast<double>(pt)) - log(static_cast<double>(fmaxf(q[t], eps))));
        }
    }
    const double total = block_sum(acc, red);
    if (threadIdx.x == 0) kl[(static_cast<size_t>(h) * 2 + dir) * gridDim.x + blockIdx.x] = total;
}

// The gradient with respect to the logits, and the loss (first workgroup).  Every workgroup adds the partial sums of its
// (head, direction) by itself, in the same order.
__global__ __launch_bounds__(kKlThreads) void train_grad_kernel(const float* __restrict__ p_v, const float* __restrict__ p_s,
                                                                 const float* __restrict__ t_v, const float* __restrict__ t_s, int n,
                                                                 int heads, float eps, const double* __restrict__ kl,
                                                                 float* __restrict__ g_v, float* __restrict__ g_s,
                                                                 float* __restrict__ loss) {
    __shared__ double red[kKlThreads / 64];
    const int h = blockIdx.y, dir = blockIdx.z, parts = gridDim.x;
    const float* __restrict__ p = (dir == 0 ? p_v : p_s) + static_cast<size_t>(h) * n;
    const float* __restrict__ q = (dir == 0 ? t_v : t_s) + static_cast<size_t>(h) * n;
    float* __restrict__ g = (dir == 0 ? g_v : g_s) + static_cast<size_t>(h) * n;
    const double* mine = kl + (static_cast<size_t>(h) * 2 + dir) * parts;
    double acc = 0.0;
    for (int i = threadIdx.x; i < parts; i += kKlThreads) acc += mine[i];
    const double total = block_sum(acc, red);
    const double inv_heads = 1.0 / heads;
#pragma unroll
    for (int i = 0; i < kKlBlock / kKlThreads; ++i) {
        const int t = blockIdx.x * kKlBlock + i * kKlThreads + threadIdx.x;
        if (t < n) {
            const float pt = p[t];
            double gt = 0.0;
            if (pt > 0.f)
                gt = static_cast<double>(pt) * (log(static_cast<double>(pt)) - log(static_cast<double>(fmaxf(q[t], eps))) - total) * inv_heads;
            g[t] = static_cast<float>(gt);
        }
    }
    if (blockIdx.x == 0 && h == 0 && dir == 0) {             // uniform over the workgroup
        double s = 0.0;
        for (size_t i = threadIdx.x; i < static_cast<size_t>(2) * heads * parts; i += kKlThreads) s += kl[i];
        const double all = block_sum(s, red);
        if (threadIdx.x == 0) *loss = static_cast<float>(all / heads);
    }
}

struct TrainParams {
    const uint16_t* kx;
    const uint16_t* vx;
    int heads, n, d_h;
    const uint16_t* w_hi;
    const uint16_t* w_lo;
    const float* b_U;
    const float* W_V;
    const float* W_S;
    const float* g_v;
    const float* g_s;
    float* part_wu;                 // [partials][256][d_h]
    float* part_vec;                // [partials][3][d_h]: dW_V, dW_S, db_U
    int chunks;                     // workgroups per 128 hidden units
    int stride;                     // partial sum c is over blocks c, c + stride, ..; a multiple of chunks
    int partials;                   // those with a block: workgroup w makes w, w + chunks, .., one after the other
};

// Matrix and vector work of a block are about equal (64 matrix instructions of 32 clocks against ~500 vector instructions
// for the 16 tokens of a lane: GELU with its slope, the logit gradients, the split into two bf16 terms), a workgroup has
// one wavefront per SIMD, and a wavefront issues in order: done one after the other, with the loads of a block waited for
// in front of it, a block took 4.7 us (8 x 32768 tokens, d_h = 256, GELU: 300 us; now 158 us, of which the issue of the ~700
// instructions of a block is the larger part; 173 while the compiler had all matrix instructions of U behind the vector instructions:
// their accumulator is pinned after each).  So the blocks are pipelined inside the wavefront: step i issues the matrix
// instructions of U for block i + 1 and of dW_U for block i - 1 and, after each of them, a piece of the activation of
// block i (scheduling barriers keep the order; pure arithmetic is pinned with empty asm statements).  The X tiles come
// straight into LDS two blocks ahead; four tile buffers.  Steps at the ends run on zeroed or stale tiles whose gradients
// are zero.
// LDS tile: 16-byte chunk c of token row r sits at chunk c ^ f(r), f(r) = 4 (r % 4) + (r / 4) % 4: 16 rows read at one chunk
// (U) hit 16 chunk positions, and 4 consecutive rows read over 64 bytes (the transposing read) hit 4 different 64-byte groups.
template <int ACT>
__global__ __launch_bounds__(kThreads, 1) void train_backward_kernel(const TrainParams p) {
    __shared__ __align__(512) unsigned char xt[kXBufs * kXTile];
    __shared__ __align__(16) float gbuf[kXBufs][2][kTokTile];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hh = lane >> 5;
    const int chunk = blockIdx.x;
    const int u = blockIdx.y * kUnitsPerWg + 32 * wave + col;      // this lane's hidden unit
    const bool active = 32 * wave + blockIdx.y * kUnitsPerWg < p.d_h;   // the wavefront's slice exists (d_h is a multiple of 64)
    const int n = p.n;

    // W_U fragments of this lane's unit: B operand of U = X W_U (lane = unit column, 8 consecutive features)
    bf16x8 whi[16], wlo[16];
    float bu = 0.f, wv = 0.f, ws = 0.f;
    if (active) {
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const size_t src = static_cast<size_t>(u) * 256 + 16 * kk + 8 * hh;
            whi[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p.w_hi + src));
            wlo[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p.w_lo + src));
        }
        bu = p.b_U[u];
        wv = p.W_V[u];
        ws = p.W_S[u];
    }
    f32x16 dwu[8];                                          // dW_U^T tile: lane (unit, hh), element 4a+c: feature 32 cb + 8a + 4hh + c
#pragma unroll
    for (int cb = 0; cb < 8; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) dwu[cb][e] = 0.f;
    float s_wv[4] = {0.f, 0.f, 0.f, 0.f}, s_ws[4] = {0.f, 0.f, 0.f, 0.f}, s_bu[4] = {0.f, 0.f, 0.f, 0.f};

    const uint32_t blocks_per_head = (n + kTokTile - 1) / kTokTile;
    const uint32_t total_blocks = static_cast<uint32_t>(p.heads) * blocks_per_head;              // < 2^31
    const int nsteps = static_cast<int>((total_blocks - chunk + p.chunks - 1) / p.chunks);       // blocks of this workgroup (>= 1)
    uint32_t next_blk = chunk, next_part = chunk;            // block that load_block() takes next, and its partial sum

    // ---- staging: a wavefront instruction deposits two token rows; wavefront w moves rows 8 w .. 8 w + 7 of a tile ----
    auto load_block = [&](int i, float& greg) __attribute__((always_inline)) {
        greg = 0.f;
        if (i >= nsteps) return;
        const uint32_t blk = next_blk;
        next_blk += p.stride;
        if (next_blk >= total_blocks) next_blk = next_part += p.chunks;
        const int head = static_cast<int>(blk / blocks_per_head);
        const int tok0 = static_cast<int>(blk - static_cast<uint32_t>(head) * blocks_per_head) * kTokTile;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row0 = 8 * wave + 2 * j, row = row0 + hh;
            const int ch = col ^ (4 * (row & 3) + ((row >> 2) & 3));
            const int tok = min(tok0 + row, n - 1);         // rows past the end: their gradients are zero
            const uint16_t* src = (ch < 16 ? p.kx : p.vx) + (static_cast<size_t>(head) * n + tok) * 128 + 8 * (ch & 15);
            lds_load16(src, xt + (i & (kXBufs - 1)) * kXTile + row0 * kXPitch);
        }
        if (wave == 0 && tok0 + col < n) greg = (hh ? p.g_s : p.g_v)[static_cast<size_t>(head) * n + tok0 + col];
    };
    // U fragment kk: row col, chunk 2 kk + hh;  dW_U fragment (cb, j): rows 16 j + 4 hh + li / 4 (+ 8), 8 bytes at feature
    // 32 cb + 16 half16 + 4 (li % 4): li of 16 lanes addresses (row li / 4, 4 features) and receives feature li of the 4 rows
    const uint32_t a_off = static_cast<uint32_t>(col * kXPitch + ((hh ^ (4 * (col & 3) + ((col >> 2) & 3))) << 4));
    const int li = lane & 15, half16 = (lane >> 4) & 1, lr = li >> 2;
    uint32_t t_off[4][2];                                   // [cb % 4][row half]
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int s = 0; s < 2; ++s)
            t_off[g][s] = static_cast<uint32_t>((8 * s + 4 * hh + lr) * kXPitch + 64 * (g ^ lr) + 16 * ((2 * half16 + ((li & 3) >> 1)) ^ (hh + 2 * s)) +
                                                8 * (li & 1));
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)xt));
    typedef __attribute__((address_space(3))) bf16x4t* lds_tr_t;
    typedef const __attribute__((address_space(3))) uint4* lds_u4_t;
    // at: this lane's address in the tile (rows are 512 bytes, tiles 512-byte aligned: the chunk number is bits 4 .. 8)
    auto read_u = [&](uint32_t at, int kk) __attribute__((always_inline)) -> bf16x8 {
        return __builtin_bit_cast(bf16x8, *(lds_u4_t)(at ^ (32u * kk)));
    };
    auto read_t = [&](const uint32_t (&at)[4][2], int cb, int j) __attribute__((always_inline)) -> bf16x8 {
        const int imm = 16 * j * kXPitch + 256 * (cb >> 2);
        const bf16x4t lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr_t)(at[cb & 3][0] + imm));
        const bf16x4t hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr_t)(at[cb & 3][1] + imm));
        bf16x8 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            r[e] = lo4[e];
            r[4 + e] = hi4[e];
        }
        return r;
    };

    for (int i = tid; i < kXBufs * kXTile / 16; i += kThreads) reinterpret_cast<uint4*>(xt)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    float g0, greg;
    load_block(0, g0);
    load_block(1, greg);
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0): also the weight fragments
    if (wave == 0) gbuf[0][hh][col] = g0;
    __syncthreads();

    // pre-activations of block i: lane (unit, hh) holds tokens 8a + 4hh + c
    f32x16 acc, acc_next, bias;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = bias[e] = bu;
    if (active) {
#pragma unroll
        for (int kk = 0; kk < 16; ++kk) {
            const bf16x8 xa = read_u(lds0 + a_off, kk);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa, whi[kk], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xa, wlo[kk], acc, 0, 0, 0);
        }
    }
    uint32_t dhi[8], dlo[8], dhi_n[8], dlo_n[8];            // pre-activation gradients (two bf16 terms) of block i - 1 and of block i
#pragma unroll
    for (int e = 0; e < 8; ++e) dhi[e] = dlo[e] = 0u;

    // blocks of partial sum c (< partials)
    auto blocks_of = [&](int c) __attribute__((always_inline)) -> int { return static_cast<int>((total_blocks - 1 - c) / p.stride) + 1; };

    constexpr int kActStages = ACT == 0 ? 7 : 16;
    constexpr int kStages = kActStages + 9;
    constexpr int kPieces = 4 * kStages;
    constexpr float kL = -1.4426950408889634f;
#define VS_PIN(x) asm volatile("" : "+v"(x))
    int part = chunk, last = blocks_of(chunk);               // the partial sum being made and the step at whose end its dW_U is complete
    for (int i = 0; i <= nsteps; ++i) {
        __builtin_amdgcn_s_waitcnt(0x0F70);                  // this wavefront's part of block i + 1 has arrived
        if (wave == 0) gbuf[(i + 1) & (kXBufs - 1)][hh][col] = greg;
        __syncthreads();
        load_block(i + 2, greg);                             // over the tile of block i - 2
        if (!active) continue;
        uint32_t ub = lds0 + ((i + 1) & (kXBufs - 1)) * kXTile + a_off, tb[4][2];
#pragma unroll
        for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                tb[g][s] = lds0 + ((i + 3) & (kXBufs - 1)) * kXTile + t_off[g][s];
                VS_PIN(tb[g][s]);
            }
        const float* const gv_at = &gbuf[i & (kXBufs - 1)][0][4 * hh];
        const float* const gs_at = &gbuf[i & (kXBufs - 1)][1][4 * hh];
        bf16x8 xu[2], xd[2];
        xu[0] = read_u(ub, 0);
        xd[0] = read_t(tb, 0, 0);
        float gv[4], gs[4], x[4], y[4], w[4], d[4], q[4];
        // piece pc: stage pc % kStages of the accumulator elements 4 g + c (tokens 8 g + 4 hh + c), g = pc / kStages
        auto piece = [&](auto pc_tag) __attribute__((always_inline)) {
            constexpr int pc = decltype(pc_tag)::value;
            constexpr int g = pc / kStages, st = pc % kStages;
            if constexpr (st == 0) {
                const float4 a = *reinterpret_cast<const float4*>(gv_at + 8 * g), b = *reinterpret_cast<const float4*>(gs_at + 8 * g);
                gv[0] = a.x; gv[1] = a.y; gv[2] = a.z; gv[3] = a.w;
                gs[0] = b.x; gs[1] = b.y; gs[2] = b.z; gs[3] = b.w;
            }
            if constexpr (st == kActStages + 6) {            // d = dpre: the first bf16 term (nearest even), two elements a word
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const f32x2 two = {d[2 * c], d[2 * c + 1]};
                    dhi_n[2 * g + c] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                    VS_PIN(dhi_n[2 * g + c]);
                }
                return;
            }
            if constexpr (st == kActStages + 8) {            // the second
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const f32x2 two = {d[2 * c], d[2 * c + 1]};
                    dlo_n[2 * g + c] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                    VS_PIN(dlo_n[2 * g + c]);
                }
                return;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if constexpr (st == 0) x[c] = acc[4 * g + c];
                if constexpr (ACT == 0) {
                    // SiLU: s = 1 / (1 + exp(-x)); z = x s; slope = s + z (1 - s).  In the end y = z, w = slope.
                    if constexpr (st == 0) { w[c] = kL * x[c]; VS_PIN(w[c]); }
                    if constexpr (st == 1) { w[c] = __builtin_amdgcn_exp2f(w[c]); VS_PIN(w[c]); }
                    if constexpr (st == 2) { w[c] = 1.f + w[c]; VS_PIN(w[c]); }
                    if constexpr (st == 3) { w[c] = __builtin_amdgcn_rcpf(w[c]); VS_PIN(w[c]); }
                    if constexpr (st == 4) { y[c] = x[c] * w[c]; VS_PIN(y[c]); }
                    if constexpr (st == 5) { q[c] = 1.f - w[c]; VS_PIN(q[c]); }
                    if constexpr (st == 6) { w[c] = fmaf(y[c], q[c], w[c]); VS_PIN(w[c]); }
                } else {
                    // GELU: z = x Phi(x), slope = Phi(x) + x phi(x), phi(x) = exp(-x^2 / 2) / sqrt(2 pi).  erf(|x| / sqrt(2)) by
                    // the rational approximation 7.1.26 of Abramowitz & Stegun (absolute error below 1.5e-7), which shares
                    // the exponential; its argument scaling and the factor 1/2 of Phi = 1/2 + erf / 2 are folded into the
                    // coefficients.  In the end y = z, w = slope.
                    if constexpr (st == 0) { d[c] = fmaf(0.23164190f, fabsf(x[c]), 1.f); VS_PIN(d[c]); }
                    if constexpr (st == 1) { w[c] = (0.5f * kL) * x[c]; VS_PIN(w[c]); }
                    if constexpr (st == 2) { w[c] = w[c] * x[c]; VS_PIN(w[c]); }
                    if constexpr (st == 3) { d[c] = __builtin_amdgcn_rcpf(d[c]); VS_PIN(d[c]); }
                    if constexpr (st == 4) { w[c] = __builtin_amdgcn_exp2f(w[c]); VS_PIN(w[c]); }
                    if constexpr (st == 5) { q[c] = fmaf(0.5f * 1.061405429f, d[c], 0.5f * -1.453152027f); VS_PIN(q[c]); }
                    if constexpr (st == 6) { q[c] = fmaf(q[c], d[c], 0.5f * 1.421413741f); VS_PIN(q[c]); }
                    if constexpr (st == 7) { q[c] = fmaf(q[c], d[c], 0.5f * -0.284496736f); VS_PIN(q[c]); }
                    if constexpr (st == 8) { q[c] = fmaf(q[c], d[c], 0.5f * 0.254829592f); VS_PIN(q[c]); }
                    if constexpr (st == 9) { q[c] = q[c] * d[c]; VS_PIN(q[c]); }
                    if constexpr (st == 10) { q[c] = fmaf(-q[c], w[c], 0.5f); VS_PIN(q[c]); }
                    if constexpr (st == 11) { q[c] = copysignf(q[c], x[c]); VS_PIN(q[c]); }
                    if constexpr (st == 12) { q[c] = 0.5f + q[c]; VS_PIN(q[c]); }                    // Phi
                    if constexpr (st == 13) { y[c] = x[c] * q[c]; VS_PIN(y[c]); }
                    if constexpr (st == 14) { x[c] = x[c] * 0.3989422804014327f; VS_PIN(x[c]); }
                    if constexpr (st == 15) { w[c] = fmaf(x[c], w[c], q[c]); VS_PIN(w[c]); }
                }
                if constexpr (st == kActStages + 0) { s_wv[c] = fmaf(gv[c], y[c], s_wv[c]); VS_PIN(s_wv[c]); }
                if constexpr (st == kActStages + 1) { s_ws[c] = fmaf(gs[c], y[c], s_ws[c]); VS_PIN(s_ws[c]); }
                if constexpr (st == kActStages + 2) { q[c] = gs[c] * ws; VS_PIN(q[c]); }
                if constexpr (st == kActStages + 3) { q[c] = fmaf(gv[c], wv, q[c]); VS_PIN(q[c]); }
                if constexpr (st == kActStages + 4) { d[c] = q[c] * w[c]; VS_PIN(d[c]); }
                if constexpr (st == kActStages + 5) { s_bu[c] += d[c]; VS_PIN(s_bu[c]); }
                if constexpr (st == kActStages + 7) {        // what the first term leaves
                    const uint32_t h = dhi_n[2 * g + (c >> 1)];
                    d[c] -= __uint_as_float((c & 1) ? (h & 0xffff0000u) : (h << 16));
                    VS_PIN(d[c]);
                }
            }
        };
        __builtin_amdgcn_sched_barrier(0);
        static_for<64>([&](auto m_tag) __attribute__((always_inline)) {
            constexpr int m = decltype(m_tag)::value;
            constexpr int k = m >> 2, part = m & 3;          // U fragment k; dW_U fragment (cb, j) = (k / 2, k % 2)
            if constexpr (part == 0) {
                if constexpr (k + 1 < 16) {
                    xu[(k + 1) & 1] = read_u(ub, k + 1);
                    xd[(k + 1) & 1] = read_t(tb, (k + 1) >> 1, (k + 1) & 1);
                }
                acc_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xu[k & 1], whi[k], k == 0 ? bias : acc_next, 0, 0, 0);
                VS_PIN(acc_next);
            } else if constexpr (part == 2) {
                acc_next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xu[k & 1], wlo[k], acc_next, 0, 0, 0);
                VS_PIN(acc_next);
            } else {
                const uint32_t* const dd = part == 1 ? dhi : dlo;
                const uint4 b4 = make_uint4(dd[4 * (k & 1)], dd[4 * (k & 1) + 1], dd[4 * (k & 1) + 2], dd[4 * (k & 1) + 3]);
                dwu[k >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xd[k & 1], __builtin_bit_cast(bf16x8, b4), dwu[k >> 1], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            constexpr int lo = (m * kPieces) / 64, hi = ((m + 1) * kPieces) / 64;
            static_for<hi - lo>([&](auto r_tag) __attribute__((always_inline)) {
                piece(std::integral_constant<int, lo + decltype(r_tag)::value>{});
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        acc = acc_next;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            dhi[e] = dhi_n[e];
            dlo[e] = dlo_n[e];
        }
        // ---- partial sums that are through: dW_U now holds the blocks up to i - 1, the vectors those up to i ----
        if (i == last) {
            uint32_t pitch = p.d_h;
            asm volatile("" : "+s"(pitch));                  // the 128 row addresses are made here, not kept over the steps
            float* const pw = p.part_wu + static_cast<size_t>(part) * 256 * pitch + u;
#pragma unroll
            for (int cb = 0; cb < 8; ++cb)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    pw[(32 * cb + 8 * (e >> 2) + 4 * hh + (e & 3)) * pitch] = dwu[cb][e];
                    dwu[cb][e] = 0.f;
                }
            part += p.chunks;
            if (part < p.partials) last += blocks_of(part);
        }
        if (i == last - 1) {                                 // (also right after the above, where the next one is a single block)
            const float t_wv = half_swap_sum((s_wv[0] + s_wv[1]) + (s_wv[2] + s_wv[3]));
            const float t_ws = half_swap_sum((s_ws[0] + s_ws[1]) + (s_ws[2] + s_ws[3]));
            const float t_bu = half_swap_sum((s_bu[0] + s_bu[1]) + (s_bu[2] + s_bu[3]));
            if (hh == 0) {
                float* const pv = p.part_vec + static_cast<size_t>(part) * 3 * p.d_h + u;
                pv[0] = t_wv;
                pv[p.d_h] = t_ws;
                pv[2 * p.d_h] = t_bu;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) s_wv[c] = s_ws[c] = s_bu[c] = 0.f;
        }
    }
#undef VS_PIN
}

// The gradients: sums of the workgroups' partial results in a fixed order, in fp64.  Outputs 0 .. 256 d_h - 1 are dW_U, then
// dW_V, dW_S, db_U.  A workgroup makes 64 outputs; its four wavefronts each add a quarter of the partials, eight loads in
// flight (one thread per output that walks all partials waits for memory 256 times over: 62 us whatever the output's
// size, four launches; now 13 us in one for 64 MB).  Bound by the memory: the partials are read once.
constexpr int kRedOut = 64;
struct TrainOuts {
    float* out[4];                                           // dW_U, dW_V, dW_S, db_U
};
__global__ __launch_bounds__(4 * kRedOut) void train_reduce_kernel(const float* __restrict__ part_wu, const float* __restrict__ part_vec,
                                                                   int partials, int d_h, TrainOuts o) {
    __shared__ double red[4][kRedOut];
    const size_t nwu = static_cast<size_t>(256) * d_h, nvec = static_cast<size_t>(3) * d_h;   // both multiples of 64
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t first = static_cast<size_t>(blockIdx.x) * kRedOut;
    const bool vec = first >= nwu;
    const float* __restrict__ src = vec ? part_vec + (first - nwu) + lane : part_wu + first + lane;
    const size_t stride = vec ? nvec : nwu;
    const int per = (partials + 3) / 4, c0 = min(per * wave, partials), c1 = min(c0 + per, partials);
    double s = 0.0;
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = src[static_cast<size_t>(c + j) * stride];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += static_cast<double>(x[j]);
    }
    for (; c < c1; ++c) s += static_cast<double>(src[static_cast<size_t>(c) * stride]);
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0) {
        const float r = static_cast<float>(((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane]);
        if (!vec) {
            o.out[0][first + lane] = r;
        } else {
            const size_t at = first - nwu + lane;
            const int which = static_cast<int>(at / d_h);
            o.out[1 + which][at - static_cast<size_t>(which) * d_h] = r;
        }
    }
}

struct TrainWs {
    size_t fwd_off, fwd_bytes, pv_off, ps_off, gv_off, gs_off, kl_off, pwu_off, pvec_off, total;
    int chunks, stride, partials, kl_parts;
};

bool dh_ok(int d_h) { return d_h >= 64 && d_h <= 1024 && d_h % 64 == 0; }

TrainWs train_ws_layout(int kv_heads, int64_t n, int d_h) {
    TrainWs w;
    const size_t rows = static_cast<size_t>(kv_heads) * n;
    const long long blocks = static_cast<long long>(kv_heads) * ((n + kTokTile - 1) / kTokTile);
    // One workgroup per compute unit over all groups of 128 hidden units (a workgroup fills its compute unit), but partial sums
    // of at most 1 / kPartials of the blocks, or kPartBlocks: a workgroup makes several, one after the other.  With one per
    // workgroup the fp32 sums were 2 (d_h = 256) to 8 times (1024) as long; 8 x 16384 tokens, SiLU / 1024: error of dW_U
    // against 64 bits 4.06e-6 (128 blocks each), 4.03e-6 now, at 394 and 456 us for the step replayed from a graph (256 d_h floats
    // more to write and add per partial sum); 8 x 32768, GELU / 256 245 and 256 us.  Below 8 blocks nothing is gained: 8 x 4096, SiLU / 1024 3.558e-6 and
    // 193 us with four blocks each, 3.560e-6 and 157 us with eight (3.569e-6 with 32).
    const int chunks = 256 / ((d_h + kUnitsPerWg - 1) / kUnitsPerWg);
    w.chunks = static_cast<int>(blocks < chunks ? blocks : chunks);
    long long want = (blocks + kPartBlocks - 1) / kPartBlocks;
    want = want < kPartials ? want : kPartials;
    w.stride = want > w.chunks ? static_cast<int>((want + w.chunks - 1) / w.chunks * w.chunks) : w.chunks;
    w.partials = static_cast<int>(blocks < w.stride ? blocks : w.stride);
    w.kl_parts = static_cast<int>((n + kKlBlock - 1) / kKlBlock);
    w.fwd_off = 0;
    w.fwd_bytes = vs::round_up(vs_index_score_workspace(kv_heads, n, d_h), 256);
    w.pv_off = w.fwd_off + w.fwd_bytes;
    w.ps_off = w.pv_off + vs::round_up(rows * 4, 256);
    w.gv_off = w.ps_off + vs::round_up(rows * 4, 256);
    w.gs_off = w.gv_off + vs::round_up(rows * 4, 256);
    w.kl_off = w.gs_off + vs::round_up(rows * 4, 256);
    w.pwu_off = w.kl_off + vs::round_up(static_cast<size_t>(kv_heads) * 2 * w.kl_parts * 8, 256);
    w.pvec_off = w.pwu_off + vs::round_up(static_cast<size_t>(w.partials) * 256 * d_h * 4, 256);
    w.total = w.pvec_off + vs::round_up(static_cast<size_t>(w.partials) * 3 * d_h * 4, 256);
    return w;
}

}  // namespace

extern "C" {

size_t vs_index_train_workspace(int kv_heads, int64_t n, int d_h) {
    if (kv_heads <= 0 || n <= 0 || n > VS_MAX_SEQ || !dh_ok(d_h)) return 0;
    return train_ws_layout(kv_heads, n, d_h).total;
}

int vs_index_train_step(const void* k_bf16, const void* v_bf16, int kv_heads, int64_t n, const vs_indexer_t* w, const float* t_v,
                        const float* t_s, float eps, float* loss, float* dW_U, float* db_U, float* dW_V, float* dW_S, void* ws,
                        size_t ws_bytes, void* stream) {
    if (!k_bf16 || !v_bf16 || !w || !t_v || !t_s || !loss || !dW_U || !db_U || !dW_V || !dW_S) return VS_ERR_INVALID_ARG;
    if (!w->W_U || !w->b_U || !w->W_V || !w->W_S) return VS_ERR_INVALID_ARG;
    if (!vs::aligned16(k_bf16) || !vs::aligned16(v_bf16)) return VS_ERR_INVALID_ARG;
    if (kv_heads <= 0 || n <= 0 || !(eps > 0.f)) return VS_ERR_INVALID_ARG;
    if (w->act != 0 && w->act != 1) return VS_ERR_INVALID_ARG;
    if (!dh_ok(w->d_h) || n > VS_MAX_SEQ || kv_heads > 65535) return VS_ERR_UNSUPPORTED;
    const TrainWs lay = train_ws_layout(kv_heads, n, w->d_h);
    if (!ws || ws_bytes < lay.total) return VS_ERR_WORKSPACE;
    if (!vs::aligned16(ws)) return VS_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned char* base = static_cast<unsigned char*>(ws);
    float* p_v = reinterpret_cast<float*>(base + lay.pv_off);
    float* p_s = reinterpret_cast<float*>(base + lay.ps_off);
    float* g_v = reinterpret_cast<float*>(base + lay.gv_off);
    float* g_s = reinterpret_cast<float*>(base + lay.gs_off);
    double* kl = reinterpret_cast<double*>(base + lay.kl_off);

    // 1. forward (the inference kernels); it leaves the split W_U in its workspace for the backward pass
    int rc = vs::index_score(k_bf16, v_bf16, kv_heads, n, w, p_v, p_s, base + lay.fwd_off, lay.fwd_bytes, stream, true);
    if (rc != VS_OK) return rc;
    const uint16_t* hi = reinterpret_cast<const uint16_t*>(base + lay.fwd_off);
    const uint16_t* lo = reinterpret_cast<const uint16_t*>(base + lay.fwd_off + vs::indexer_split_lo_offset(w->d_h));
    // 2. loss and logit gradients
    const dim3 kl_grid(lay.kl_parts, kv_heads, 2);
    hipLaunchKernelGGL(train_kl_kernel, kl_grid, dim3(kKlThreads), 0, st, p_v, p_s, t_v, t_s, static_cast<int>(n), eps, kl);
    VS_LAUNCH_CHECK();
    hipLaunchKernelGGL(train_grad_kernel, kl_grid, dim3(kKlThreads), 0, st, p_v, p_s, t_v, t_s, static_cast<int>(n), kv_heads, eps, kl,
                       g_v, g_s, loss);
    VS_LAUNCH_CHECK();
    // 3. backward
    TrainParams p{};
    p.kx = static_cast<const uint16_t*>(k_bf16);
    p.vx = static_cast<const uint16_t*>(v_bf16);
    p.heads = kv_heads;
    p.n = static_cast<int>(n);
    p.d_h = w->d_h;
    p.w_hi = hi;
    p.w_lo = lo;
    p.b_U = w->b_U;
    p.W_V = w->W_V;
    p.W_S = w->W_S;
    p.g_v = g_v;
    p.g_s = g_s;
    p.part_wu = reinterpret_cast<float*>(base + lay.pwu_off);
    p.part_vec = reinterpret_cast<float*>(base + lay.pvec_off);
    p.chunks = lay.chunks;
    p.stride = lay.stride;
    p.partials = lay.partials;
    const dim3 grid(lay.chunks, (w->d_h + kUnitsPerWg - 1) / kUnitsPerWg);
    if (w->act == 0) hipLaunchKernelGGL(train_backward_kernel<0>, grid, dim3(kThreads), 0, st, p);
    else hipLaunchKernelGGL(train_backward_kernel<1>, grid, dim3(kThreads), 0, st, p);
    VS_LAUNCH_CHECK();
    const TrainOuts outs{{dW_U, dW_V, dW_S, db_U}};
    hipLaunchKernelGGL(train_reduce_kernel, dim3(static_cast<unsigned>(259 * w->d_h / kRedOut)), dim3(4 * kRedOut), 0, st, p.part_wu,
                       p.part_vec, lay.partials, w->d_h, outs);
    VS_LAUNCH_CHECK();
    return VS_OK;
}

}  // extern "C"
