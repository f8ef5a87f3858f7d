// Backward pass of the sparse causal attention, for gfx950 (bf16 MFMA).
//
// The student is trained through the attention of TalkingMachines Sec. 4.2,
// O = softmax(scale * Q K^T) V over each query's allowed key set
// {c_0, c_{a-W}, ..., c_a}. Given dO, the chain rule over the masked row
// softmax gives, with P recomputed from the forward's log-sum-exp:
//
//   delta_i = rowsum(dO_i * O_i)          (= rowsum(P_i * dP_i))
//   dP = dO V^T,  dS = P * (dP - delta)
//   dV = P^T dO,  dQ = scale dS K,  dK = scale dS^T Q
//
// Three kernels, all on the whole-sequence layout [B, L, H, D] (and
// bwd_sum_kernel, which adds up the parts of split tiles):
// - bwd_delta_kernel: delta [B, H, L] in fp32;
// - bwd_dq_kernel: one workgroup of 4 waves per 128-row query tile (tiles
//   never straddle a chunk, so a tile's rows share their key ranges); per
//   64-key tile, loaded straight into LDS while the previous tile computes,
//   it recomputes S^T = K Q^T and dP^T = V dO^T and accumulates
//   dQ^T += K^T dS^T, the same operand layouts as the forward's
//   O^T += V^T P^T with row-major V (K^T read with transposing LDS reads);
// - bwd_dkdv_kernel: one workgroup of 4 waves per 128-key tile of one chunk
//   (two workgroups share a CU, so each SIMD runs two independent waves);
//   the queries that see a key chunk c form one range (all of them for c_0,
//   chunks c .. c+W otherwise); per 32-query stage, loaded straight into LDS
//   while the previous stage computes, it forms S = Q K^T and dP = dO V^T
//   (one key per lane) and accumulates dV^T += dO^T P and dK^T += Q^T dS,
//   with dO^T and Q^T read with transposing LDS reads. The c_0 tiles, which
//   see every query, are dispatched first.
// P and dS are rounded to bf16 for the MFMAs; accumulation is fp32; results
// are rounded to bf16 once. No atomics: the result is deterministic.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "tm_device.h"
#include "tm_internal.h"

namespace tmk {
namespace {

constexpr int kDqThreads = 256;    // 4 waves: 128 query rows; two workgroups per CU
constexpr int kDkdvThreads = 256;  // 4 waves: 128 keys; two workgroups per CU

typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
typedef __attribute__((address_space(3))) bf16x4_t lds_bf16x4_t;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4_t;

// LDS tiles of both gradient kernels (K and V in dQ; Q, dO and V in dK/dV)
// put 16-byte chunk c of row `row` at c ^ tr_swizzle<D>(row).
// Per-lane LDS byte offsets inside such a tile (rows at multiples of 16 keep
// the pattern):
// - row operand (A of S^T = K Q^T, or A of S = Q K^T): row l32, chunk
//   2*kk + hw, for k-step kk: row(kk);
// - transposed operand (A of X^T-times-P products over 16 rows per step):
//   two transposing reads, tr_lo(d) and tr_hi(d), of rows 4*hw + gi/4 and
//   + 8 at element columns 32*d + 16*(grp & 1) + 4*(gi & 3); with these the
//   MFMA's k index e of a lane runs over rows 4*hw + e%4 + 8*(e/4), matching
//   the natural output layout of the first product (register i of a lane:
//   row 8*(i/4) + 4*hw + i%4).
// The chunk is 2*kk + hw or 4*d + cbase, and the swizzle's XOR only touches
// the chunk bits, so row(kk) = row0 ^ (kk << 5) and tr_lo(d) = tr0 ^ (d << 6):
// three registers instead of sixteen. pinned() and at() make a stage derive them anew
// (one XOR per use) rather than have the compiler keep all of them.
template <int D>
struct TileBases {
    static constexpr int ROWB = D * 2;
    uint32_t row0, tr0, tr8;
    __device__ __forceinline__ TileBases(int lane) {
        const int l32 = lane & 31, hw = lane >> 5;
        row0 = l32 * ROWB + ((hw ^ tr_swizzle<D>(l32)) << 4);
        const int grp = lane >> 4, gi = lane & 15;
        const int r = 4 * hw + (gi >> 2);
        const int cbase = 2 * (grp & 1) + ((gi & 3) >> 1);
        const int half = (gi & 1) * 8;
        tr0 = r * ROWB + ((cbase ^ tr_swizzle<D>(r)) << 4) + half;
        tr8 = r * ROWB + ((cbase ^ tr_swizzle<D>(r + 8)) << 4) + half;
    }
    __device__ __forceinline__ TileBases pinned() const { return at(0); }
    // The same in the tile at LDS offset `base` (a multiple of 1 KB, which the
    // XORs leave alone).
    __device__ __forceinline__ TileBases at(uint32_t base) const {
        TileBases t = *this;
        t.row0 += base;
        t.tr0 += base;
        t.tr8 += base;
        asm volatile("" : "+v"(t.row0), "+v"(t.tr0), "+v"(t.tr8));
        return t;
    }
    __device__ __forceinline__ uint32_t row(int kk) const { return row0 ^ (kk << 5); }
    __device__ __forceinline__ uint32_t tr_lo(int d) const { return tr0 ^ (d << 6); }
    __device__ __forceinline__ uint32_t tr_hi(int d) const { return (tr8 ^ (d << 6)) + 8 * ROWB; }
};

template <int D>
__device__ __forceinline__ bf16x8_t read_tr(const lds_u8* tile, uint32_t lo, uint32_t hi) {
    const bf16x4_t a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(tile + lo));
    const bf16x4_t b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(tile + hi));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Stores a wave's 32 rows of D bf16, held as X^T accumulators (register 4*g + e
// of block d in a lane: row l32, dimension 32*d + 8*g + 4*hw + e), scaled, as
// whole rows: through 32 * D * 2 bytes of the wave's own LDS (16-byte chunk c
// of row r at c ^ (r & CM)), so that a store instruction covers whole rows and
// not 8 bytes of 32 of them. Rows at or past n are not stored.
template <int D>
__device__ __forceinline__ void store_rows(lds_u8* rows, const f32x16_t (&acc)[D / 32], float scale,
                                           __bf16* out, int64_t stride, int n, int lane) {
    constexpr int ROWB = D * 2, CPR = D / 8, CM = CPR < 16 ? 7 : 15;
    const int l32 = lane & 31, hw = lane >> 5;
#pragma unroll
    for (int d = 0; d < D / 32; ++d) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4_t w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(acc[d][4 * g + e] * scale);
            *(lds_bf16x4_t*)(rows + l32 * ROWB + (((4 * d + g) ^ (l32 & CM)) << 4) + 8 * hw) = w;
        }
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 32 * CPR / 64; ++i) {
        const int ch = 64 * i + lane, row = ch / CPR;
        const f32x4_t w = *(const lds_f32x4_t*)(rows + row * ROWB + (((ch % CPR) ^ (row & CM)) << 4));
        if (row < n) *reinterpret_cast<f32x4_t*>(out + row * stride + (ch % CPR) * 8) = w;
    }
}

// The same accumulators unscaled, in register order: whole KBs per store.
template <int D>
__device__ __forceinline__ void store_part(float* part, const f32x16_t (&acc)[D / 32], int lane) {
#pragma unroll
    for (int d = 0; d < D / 32; ++d)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<f32x4_t*>(part + (4 * d + g) * 256 + 4 * lane) =
                f32x4_t{acc[d][4 * g], acc[d][4 * g + 1], acc[d][4 * g + 2], acc[d][4 * g + 3]};
}

// ---------------------------------------------------------------------------
// delta = rowsum(dO * O): D / 8 lanes per (batch, token, head) row, 16 bytes
// each, one workgroup per head and 64 tokens, so that both tensors are read in
// whole rows and delta is written in runs of 64 floats. Bound by HBM: 0.68 GB at
// 480p, 40 heads, 21 frames in 119 us (5.7 TB/s; 174 us with one thread per row).
// ---------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void bwd_delta_kernel(const __bf16* __restrict__ o,
                                                        const __bf16* __restrict__ dout,
                                                        float* __restrict__ delta, int B, int L,
                                                        int H) {
    constexpr int LPR = D / 8;         // lanes per row
    constexpr int RPP = 256 / LPR;     // rows per pass
    constexpr int PASSES = 64 / RPP;
    __shared__ float sums[64];
    const int blocks = (L + 63) / 64;
    // consecutive workgroups take the heads of the same tokens: their rows are
    // neighbours in memory
    const int h = blockIdx.x % H;
    const int rest = blockIdx.x / H;
    const int t0 = rest % blocks * 64;
    const int64_t b = rest / blocks;
    const int c = threadIdx.x % LPR, r0 = threadIdx.x / LPR;
    bf16x8_t a[PASSES], g[PASSES];
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        const int64_t row = (b * L + min(t0 + i * RPP + r0, L - 1)) * H + h;
        a[i] = *reinterpret_cast<const bf16x8_t*>(o + row * D + c * 8);
        g[i] = *reinterpret_cast<const bf16x8_t*>(dout + row * D + c * 8);
    }
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc = fmaf(static_cast<float>(a[i][e]), static_cast<float>(g[i][e]), acc);
#pragma unroll
        for (int m = 1; m < LPR; m *= 2) acc += __shfl_xor(acc, m);
        if (c == 0) sums[i * RPP + r0] = acc;
    }
    __syncthreads();
    const int t = t0 + static_cast<int>(threadIdx.x);
    if (threadIdx.x < 64 && t < L) delta[(b * H + h) * L + t] = sums[threadIdx.x];
}

// Key ranges of query chunk a: c_0, and chunks max(1, a - W) .. a, merged.
struct Ranges {
    int n;
    int b0, e0, b1, e1;
};
__device__ __forceinline__ Ranges key_ranges(const BwdArgs& a, int chunk) {
    Ranges r;
    const int ref_end = min(a.ref_tok, a.L);
    if (chunk == 0) {
        r.n = 1;
        r.b0 = 0;
        r.e0 = ref_end;
        return r;
    }
    const int lo_chunk = max(1, chunk - a.window);
    const int b1 = a.ref_tok + (lo_chunk - 1) * a.chunk_tok;
    const int e1 = min(a.ref_tok + chunk * a.chunk_tok, a.L);
    if (b1 <= ref_end) {
        r.n = 1;
        r.b0 = 0;
        r.e0 = e1;
    } else {
        r.n = 2;
        r.b0 = 0;
        r.e0 = ref_end;
        r.b1 = b1;
        r.e1 = e1;
    }
    return r;
}

// Chunk of tile t of a chunk-aligned tiling (ref_tiles tiles for c_0, then
// chunk_tiles per chunk), its first row and its row end.
__device__ __forceinline__ void tile_rows(const BwdArgs& a, int t, int BM, int ref_tiles, int chunk_tiles,
                                          int& chunk, int& r0, int& r1) {
    if (t < ref_tiles) {
        chunk = 0;
        r0 = t * BM;
        r1 = min(r0 + BM, min(a.ref_tok, a.L));
    } else {
        chunk = 1 + (t - ref_tiles) / chunk_tiles;
        const int j = (t - ref_tiles) % chunk_tiles;
        const int cs = a.ref_tok + (chunk - 1) * a.chunk_tok;
        r0 = cs + j * BM;
        r1 = min(min(r0 + BM, cs + a.chunk_tok), a.L);
    }
}

// ---------------------------------------------------------------------------
// dQ: per 128-row query tile, over its key ranges in 64-key tiles
// ---------------------------------------------------------------------------
// Each wave owns 32 query rows and holds their Q and dO fragments (the B
// operands of S^T = K Q^T and dP^T = V dO^T) and their dQ^T accumulators in
// registers. The key tiles of the tile's (at most two) key ranges form one
// sequence; each tile's K and V rows arrive by direct global->LDS loads into
// two alternating buffers, the next tile's loads in flight during the current
// tile's arithmetic; one barrier per tile.
template <int D>
__global__ __launch_bounds__(kDqThreads, 2) void bwd_dq_kernel(const BwdArgs a) {
    constexpr int ROWB = D * 2, KK = D / 16, DB = D / 32, CPR = D / 8;
    constexpr int BM = kBwdQTile, BN = 64;
    constexpr int NW = kDqThreads / 64;         // waves
    constexpr int KT = BN * ROWB;               // one tensor's key tile in LDS
    constexpr int BUF = 2 * KT;                 // K tile, then V tile
    constexpr int NBW = KT / 1024 / NW;         // 1-KB direct loads per wave, tensor and tile
    static_assert(NBW >= 1 && NBW * NW * 1024 == KT, "key tile must split over the waves");
    static_assert(BM == NW * 32, "32 query rows per wave");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * BUF];
    lds_u8* const L = (lds_u8*)smem;
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(L));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hw = lane >> 5;
    // The chunks' query tiles (which see c_0 and W + 1 chunks of keys) first,
    // grouped per XCD so that a head's tiles share an L2; c_0's tiles (which
    // see c_0 only) last, in plain dispatch order, so that they spread over
    // the XCDs and fill the end of the grid.
    const int BH = a.B * a.H;
    const int rest = a.q_tiles - a.q_ref_tiles;
    const int n_chunk = rest * BH * a.q_parts;
    int bh, t, part;
    if (static_cast<int>(blockIdx.x) < n_chunk) {
        int id = xcd_logical_id(blockIdx.x, n_chunk);
        part = id % a.q_parts;
        id /= a.q_parts;
        bh = id / rest;
        t = a.q_ref_tiles + id % rest;
    } else {
        int r = blockIdx.x - n_chunk;
        part = r % a.q_parts;
        r /= a.q_parts;
        bh = r / a.q_ref_tiles;
        t = r % a.q_ref_tiles;
    }
    const int h = bh % a.H, b = bh / a.H;
    int chunk, q0, q1;
    tile_rows(a, t, BM, a.q_ref_tiles, a.q_chunk_tiles, chunk, q0, q1);
    if (q0 >= q1) return;  // a tile past the end of a short last chunk

    const int64_t st = static_cast<int64_t>(a.H) * D;
    const int64_t base = static_cast<int64_t>(b) * a.L * st + h * D;
    const __bf16* qg = static_cast<const __bf16*>(a.q) + base;
    const __bf16* kg = static_cast<const __bf16*>(a.k) + base;
    const __bf16* vg = static_cast<const __bf16*>(a.v) + base;
    const __bf16* dog = static_cast<const __bf16*>(a.dout) + base;
    const float* lse = a.lse + (static_cast<int64_t>(b) * a.H + h) * a.L;
    const float* dl = a.delta + (static_cast<int64_t>(b) * a.H + h) * a.L;

    // key tile j of the sequence: first key k0 and end ke of its range
    const Ranges rg = key_ranges(a, chunk);
    const int n0 = (rg.e0 - rg.b0 + BN - 1) / BN;
    const int tiles = n0 + (rg.n == 2 ? (rg.e1 - rg.b1 + BN - 1) / BN : 0);
    // this part's tiles [j0, nt) (none where there are fewer tiles than parts)
    const int j0 = tiles * part / a.q_parts, nt = tiles * (part + 1) / a.q_parts;
    auto tile_at = [&](int j, int& k0, int& ke) __attribute__((always_inline)) {
        if (j < n0) {
            k0 = rg.b0 + j * BN;
            ke = rg.e0;
        } else {
            k0 = rg.b1 + (j - n0) * BN;
            ke = rg.e1;
        }
    };
    // Direct loads of key tile j into buffer u (rows past ke repeat row
    // ke - 1: finite values, masked below), swizzled as in the dK/dV kernel.
    auto issue = [&](int j, int u) __attribute__((always_inline)) {
        int k0, ke;
        tile_at(j, k0, ke);
        const int last = ke - 1 - k0;
        // per-lane terms derived anew per tile, not kept (spilled) across it
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const void* ks = uniform_ptr(kg + k0 * st);
        const void* vs = uniform_ptr(vg + k0 * st);
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            const int blk = i * NW + wave;
            const int ch = blk * 64 + ln;
            const int row = ch / CPR;
            const int gc = (ch % CPR) ^ tr_swizzle<D>(row);
            const uint32_t voff = static_cast<uint32_t>((min(row, last) * st + gc * 8) * 2);
            const uint32_t l = lds_base + u * BUF + blk * 1024;
            lds_dma16x2(ks, voff, l, vs, voff, l + KT);
        }
    };

    // the first tile's loads, and behind them this wave's operands: both
    // latencies pass together
    if (j0 < nt) issue(j0, 0);
    // this wave's 32 query rows: Q and dO as the B operands of S^T and dP^T
    const int qrow = q0 + wave * 32 + l32;
    const int qr = min(qrow, q1 - 1);
    bf16x8_t qf[KK], dof[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        qf[kk] = *reinterpret_cast<const bf16x8_t*>(qg + qr * st + kk * 16 + hw * 8);
        dof[kk] = *reinterpret_cast<const bf16x8_t*>(dog + qr * st + kk * 16 + hw * 8);
    }
    const float lse2 = lse[qr] * 1.4426950408889634f;
    const float dlt = dl[qr];
    const float c = a.scale_log2;
    const TileBases<D> tb(lane);
    f32x16_t acc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d] = f32x16_t{};

    // Key tile j from buffer u: S^T = K Q^T and dP^T = V dO^T per 32-key
    // block kb (register i: key 32*kb + 8*(i/4) + 4*hw + i%4, query l32),
    // dS^T as the B operand of dQ^T += K^T dS^T (k-step = 16 keys). Keys past
    // the range, which only its last tile can hold, get a score of -inf.
    auto compute = [&](int u, int j) __attribute__((always_inline)) {
        int k0, ke;
        tile_at(j, k0, ke);
        const lds_u8* Ks = L;
        const lds_u8* Vs = Ks + KT;
        const TileBases<D> off = tb.at(u * BUF);
        // The tile's MFMAs in one order: S(kb 0), dP(0), S(1), dP(1), then dQ,
        // each preceded by the LDS read of the operand RING MFMAs ahead and
        // followed by its share of the arithmetic of what is complete by then:
        // P(0) under dP(0), dS(0) under S(1) and dP(1), P(1) under dP(1), dS(1)
        // under the first half of dQ (a wave hides its arithmetic under its
        // own MFMAs, far less under the other wave's). With the arithmetic in
        // lumps and the accumulators moved between a masked and an unmasked
        // copy of this body, dQ of the 480p clip took 8.22 ms, now 8.09.
        constexpr int RING = 4, NS = 4 * KK, NT = NS + 4 * DB;
        constexpr int EP = 16 / KK;  // elements per step
        auto frag = [&](int m) __attribute__((always_inline)) {
            if (m < NS) {
                const lds_u8* T = (m / KK) % 2 == 0 ? Ks : Vs;
                return *(const lds_bf16x8_t*)(T + (m / (2 * KK)) * 32 * ROWB + off.row(m % KK));
            }
            const int j4 = (m - NS) / DB, d = (m - NS) % DB;
            return read_tr<D>(Ks + 16 * j4 * ROWB, off.tr_lo(d), off.tr_hi(d));
        };
        bf16x8_t pf[4], fr[RING];
        f32x16_t s[2], dp[2];
        s[0] = s[1] = dp[0] = dp[1] = f32x16_t{};
        // P of element i of key block kb, in place of its score; dS from it
        auto form_p = [&](int kb, int i) __attribute__((always_inline)) {
            s[kb][i] = __builtin_amdgcn_exp2f(fmaf(s[kb][i], c, -lse2));
        };
        auto form_ds = [&](int kb, int i) __attribute__((always_inline)) {
            pf[2 * kb + i / 8][i % 8] = static_cast<__bf16>(s[kb][i] * (dp[kb][i] - dlt));
        };
#pragma unroll
        for (int m = 0; m < RING; ++m) fr[m] = frag(m);
        auto step = [&](int m) __attribute__((always_inline)) {
            const int kb = m / (2 * KK), kk = m % KK;
            if (m >= NS) {
                const int j4 = (m - NS) / DB, d = (m - NS) % DB;
                acc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], pf[j4], acc[d], 0, 0, 0);
            } else if ((m / KK) % 2 == 0) {
                s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], qf[kk], s[kb], 0, 0, 0);
            } else {
                dp[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], dof[kk], dp[kb], 0, 0, 0);
            }
            if (m + RING < NT) fr[m % RING] = frag(m + RING);
            if ((m == KK || m == 3 * KK) && k0 + BN > ke) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + 32 * kb + 8 * (i / 4) + 4 * hw + (i % 4) >= ke) s[kb][i] = kNegInf;
            }
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int e0 = (m - (2 * b + 1) * KK) * EP;  // P: S(b) is complete
                const int d0 = (m - (2 * b + 2) * KK) * EP;  // dS: dP(b) is complete
#pragma unroll
                for (int e = 0; e < EP; ++e) {
                    if (e0 + e >= 0 && e0 + e < 16) form_p(b, e0 + e);
                    if (d0 + e >= 0 && d0 + e < 16) form_ds(b, d0 + e);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        // (three loops, as the compiler does not unroll all steps as one)
#pragma unroll
        for (int m = 0; m < 2 * KK; ++m) step(m);
#pragma unroll
        for (int m = 2 * KK; m < NS; ++m) step(m);
#pragma unroll
        for (int m = NS; m < NT; ++m) step(m);
    };
    wait_lds_dma();
    __syncthreads();
    // One body for both buffers: with a copy per buffer, leaving the loop
    // between them made the compiler move the accumulators on every tile.
    for (int j = j0, u = 0; j < nt; ++j, u ^= 1) {
        // buffer u ^ 1 was last read in the previous tile, before the barrier
        if (j + 1 < nt) issue(j + 1, u ^ 1);
        compute(u, j);
        wait_lds_dma();
        __syncthreads();
    }

    // (every wave is past the last tile's barrier: the LDS is free)
    const int w0 = q0 + wave * 32;
    if (w0 < q1) {
        if (a.q_parts > 1) {
            const int64_t at = ((static_cast<int64_t>(bh) * a.q_tiles + t) * a.q_parts + part) * NW + wave;
            store_part<D>(a.dq_part + at * (32 * D), acc, lane);
        } else {
            store_rows<D>(L + wave * 32 * ROWB, acc, a.scale, static_cast<__bf16*>(a.dq) + base + w0 * st, st,
                          q1 - w0, lane);
        }
    }
}

// ---------------------------------------------------------------------------
// dK, dV: per 128-key tile of one chunk, over the queries that see the chunk
// ---------------------------------------------------------------------------
// Each wave owns 32 keys and holds their K fragments (the B operand of
// S = Q K^T) and their dK^T and dV^T accumulators in registers (256 per lane at
// D = 128, so two waves fit on a SIMD); the workgroup's V rows (the B operand of
// dP = dO V^T) sit in LDS. The 32-query stages of Q, dO, lse and delta arrive
// by direct global->LDS loads into two alternating buffers, the next stage's
// loads in flight during the current stage's arithmetic; one barrier per
// stage. Two workgroups per CU keep the SIMDs' two waves out of step, so that
// one wave's softmax arithmetic can overlap the other's MFMAs (partly: two
// waves that both alternate the two kinds of work overlap only in part).
template <int D>
__global__ __launch_bounds__(kDkdvThreads, 2) void bwd_dkdv_kernel(const BwdArgs a) {
    constexpr int ROWB = D * 2, KK = D / 16, DB = D / 32, CPR = D / 8;
    constexpr int BQ = 32;                      // queries per stage
    constexpr int NW = kDkdvThreads / 64;       // waves
    constexpr int TILE = BQ * ROWB;             // one tensor's stage tile in LDS
    constexpr int STAGE = 2 * TILE;             // Q tile, then dO tile
    constexpr int NB = TILE / 1024;             // 1-KB direct loads per tensor and stage
    static_assert(NB % NW == 0, "stage tile must split over the waves");
    constexpr int VEC = 2 * STAGE;              // lse and delta: 2 buffers x 64 floats each
    constexpr int VT = VEC + 4 * 256;           // V rows of the workgroup's keys
    static_assert(kBwdKTile == NW * 32, "32 keys per wave");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[VT + kBwdKTile * ROWB];
    lds_u8* const L = (lds_u8*)smem;
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(L));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hw = lane >> 5;
    // c_0's key tiles (every query sees them: 3.5x the work of a chunk's
    // tile at W = 1) of all heads first, in plain dispatch order so that they
    // spread over the 8 XCDs (grouping them per XCD would leave one XCD with
    // all of them); the chunks' tiles after them, grouped per XCD so that a
    // head's tiles share an L2.
    const int BH = a.B * a.H;
    const int n_ref = a.k_ref_tiles * BH * a.k_ref_parts;
    int bh, t, part, parts;
    int64_t slot = 0;  // of this part's sums
    if (static_cast<int>(blockIdx.x) < n_ref) {
        parts = a.k_ref_parts;
        slot = blockIdx.x;
        int r = blockIdx.x;
        part = r % parts;
        r /= parts;
        bh = r / a.k_ref_tiles;
        t = r % a.k_ref_tiles;
    } else {
        const int rest = a.k_tiles - a.k_ref_tiles;
        parts = a.k_chunk_parts;
        int id = xcd_logical_id(blockIdx.x - n_ref, rest * BH * parts);
        slot = (a.k_ref_parts > 1 ? n_ref : 0) + id;
        part = id % parts;
        id /= parts;
        bh = id / rest;
        t = a.k_ref_tiles + id % rest;
    }
    const int h = bh % a.H, b = bh / a.H;
    int chunk, k0, k1;
    tile_rows(a, t, kBwdKTile, a.k_ref_tiles, a.k_chunk_tiles, chunk, k0, k1);
    if (k0 >= k1) return;
    // queries [qbeg, qend) see key chunk `chunk`
    int qbeg, qend;
    if (chunk == 0) {
        qbeg = 0;
        qend = a.L;
    } else {
        qbeg = a.ref_tok + (chunk - 1) * a.chunk_tok;
        qend = min(a.ref_tok + (chunk + a.window) * a.chunk_tok, a.L);
    }
    // this part's 32-query stages (none where there are fewer stages than parts)
    int n_st = (qend - qbeg + BQ - 1) / BQ;
    {
        const int s0 = n_st * part / parts, s1 = n_st * (part + 1) / parts;
        qend = min(qbeg + s1 * BQ, qend);
        qbeg += s0 * BQ;
        n_st = s1 - s0;
    }

    const int64_t st = static_cast<int64_t>(a.H) * D;
    const int64_t base = static_cast<int64_t>(b) * a.L * st + h * D;
    const __bf16* qg = static_cast<const __bf16*>(a.q) + base;
    const __bf16* kg = static_cast<const __bf16*>(a.k) + base;
    const __bf16* vg = static_cast<const __bf16*>(a.v) + base;
    const __bf16* dog = static_cast<const __bf16*>(a.dout) + base;
    const float* lse = a.lse + (static_cast<int64_t>(b) * a.H + h) * a.L;
    const float* dl = a.delta + (static_cast<int64_t>(b) * a.H + h) * a.L;

    // Direct loads of the stage starting at query q0 into buffer u: rows past
    // qend repeat row qend - 1 (finite values; seal() below zeroes their P
    // and dS). Each 1-KB block
    // holds 64 consecutive 16-byte LDS chunks of the swizzled tile; the lane
    // whose chunk is logical chunk gc of row `row` fetches that chunk.
    auto issue = [&](int q0, int u) __attribute__((always_inline)) {
        const int last = qend - 1 - q0;
        const void* qs = uniform_ptr(qg + q0 * st);
        const void* ds = uniform_ptr(dog + q0 * st);
#pragma unroll
        for (int i = 0; i < NB / NW; ++i) {
            const int blk = i * NW + wave;
            const int ch = blk * 64 + lane;
            const int row = ch / CPR;
            const int gc = (ch % CPR) ^ tr_swizzle<D>(row);
            const uint32_t voff = static_cast<uint32_t>((min(row, last) * st + gc * 8) * 2);
            const uint32_t l = lds_base + u * STAGE + blk * 1024;
            lds_dma16x2(qs, voff, l, ds, voff, l + TILE);
        }
        if (wave == NW - 1) {
            const uint32_t vo = static_cast<uint32_t>(min(lane, last) * 4);
            lds_dma4x2(uniform_ptr(lse + q0), vo, lds_base + VEC + u * 256, uniform_ptr(dl + q0), vo,
                       lds_base + VEC + 512 + u * 256);
        }
    };

    // the first stage's loads; the K and V rows' latency passes with theirs
    if (n_st > 0) issue(qbeg, 0);
    // this wave's keys: k0 + 32 * wave + l32
    const int kw = k0 + 32 * wave;
    const bool busy = kw < k1;
    bf16x8_t kf[KK];
    {
        const int kr = min(kw + l32, k1 - 1);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            kf[kk] = *reinterpret_cast<const bf16x8_t*>(kg + kr * st + kk * 16 + hw * 8);
    }
    // this wave's 32 V rows into LDS (rows past k1 repeat row k1 - 1)
    {
        const int vk = min(kw, k1 - 1);
        const void* vs = uniform_ptr(vg + static_cast<int64_t>(vk) * st);
        const int vlast = k1 - 1 - vk;
#pragma unroll
        for (int i = 0; i < 32 * ROWB / 1024; i += 2) {
            uint32_t vo[2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int ch = (i + m) * 64 + lane;
                const int row = ch / CPR;
                const int gc = (ch % CPR) ^ tr_swizzle<D>(row);
                vo[m] = static_cast<uint32_t>((min(row, vlast) * st + gc * 8) * 2);
            }
            const uint32_t l = lds_base + VT + wave * 32 * ROWB + i * 1024;
            lds_dma16x2(vs, vo[0], l, vs, vo[1], l + 1024);
        }
    }
    const TileBases<D> tb(lane);
    f32x16_t dk[DB], dv[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) dk[d] = dv[d] = f32x16_t{};
    const float c = a.scale_log2;

    // One stage from buffer U: S = Q K^T and dP = dO V^T (register i: query
    // 8*(i/4) + 4*hw + i%4 of the stage, key l32 of the wave), then
    // dV^T += dO^T P and dK^T += Q^T dS over the stage's 32 queries.
    auto compute = [&](auto ucst, int q0) __attribute__((always_inline)) {
        constexpr int U = decltype(ucst)::value;
        const lds_u8* Qb = L + U * STAGE;
        const lds_u8* Db = Qb + TILE;
        const lds_u8* Vw = L + VT + wave * 32 * ROWB;
        const lds_f32* ls = (const lds_f32*)(L + VEC + U * 256);
        const lds_f32* dls = (const lds_f32*)(L + VEC + 512 + U * 256);
        const TileBases<D> off = tb.pinned();
        // The stage's MFMAs in one order: S, dP, dV, dK, each preceded by the
        // LDS reads of the operands some MFMAs ahead and followed by its share
        // of the arithmetic of what is complete by then: P under dP, dS under dV
        // (dK/dV of the 480p clip, 40 heads: 10.99 ms with S and dP alternating
        // and the arithmetic after both, 10.69 so).
        constexpr int RING = 4, VRING = 3, NT = 2 * KK + 4 * DB;
        constexpr int EP = 16 / KK;              // elements per step
        constexpr int P0 = KK + KK / 4;          // first step of P
        constexpr int D0 = 2 * KK + KK / 4;      // first step of dS
        auto frag = [&](int m) __attribute__((always_inline)) {
            if (m < KK) return *(const lds_bf16x8_t*)(Qb + off.row(m));
            if (m < 2 * KK) return *(const lds_bf16x8_t*)(Db + off.row(m - KK));
            const int n = (m - 2 * KK) % (2 * DB), j = n / DB, d = n % DB;
            return read_tr<D>((m < 2 * KK + 2 * DB ? Db : Qb) + 16 * j * ROWB, off.tr_lo(d), off.tr_hi(d));
        };
        f32x16_t s = f32x16_t{}, dp = f32x16_t{};
        bf16x8_t fr[RING], vb[VRING], pf[2], sf[2];
        f32x4_t x, y;  // lse (+inf for rows past qend, so that P = 0) and delta of four queries
#pragma unroll
        for (int m = 0; m < RING; ++m) fr[m] = frag(m);
#pragma unroll
        for (int m = 0; m < NT; ++m) {
            const int n = (m - 2 * KK) % (2 * DB), j = n / DB, d = n % DB;
            if (m < KK) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], kf[m], s, 0, 0, 0);
            else if (m < 2 * KK)
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], vb[(m - KK) % VRING], dp, 0, 0, 0);
            else if (m < 2 * KK + 2 * DB)
                dv[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], pf[j], dv[d], 0, 0, 0);
            else dk[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[m % RING], sf[j], dk[d], 0, 0, 0);
            if (m + RING < NT) fr[m % RING] = frag(m + RING);
            const int kv = m + VRING - KK;  // V operand read VRING MFMAs ahead
            if (kv >= 0 && kv < KK) vb[kv % VRING] = *(const lds_bf16x8_t*)(Vw + off.row(kv));
#pragma unroll
            for (int e = 0; e < EP; ++e) {
                const int ip = (m - P0) * EP + e, id = (m - D0) * EP + e;
                if (ip >= 0 && ip < 16) {
                    s[ip] = __builtin_amdgcn_exp2f(fmaf(s[ip], c, -(x[ip % 4] * 1.4426950408889634f)));
                    pf[ip / 8][ip % 8] = static_cast<__bf16>(s[ip]);
                }
                if (id >= 0 && id < 16) sf[id / 8][id % 8] = static_cast<__bf16>(s[id] * (dp[id] - y[id % 4]));
            }
            // the next step's lse or delta, when it starts a group of four queries
            const int np = (m + 1 - P0) * EP, nd = (m + 1 - D0) * EP;
            if (np >= 0 && np < 16 && np % 4 == 0) x = *(const lds_f32x4_t*)(ls + 2 * np + 4 * hw);
            if (nd >= 0 && nd < 16 && nd % 4 == 0) y = *(const lds_f32x4_t*)(dls + 2 * nd + 4 * hw);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // The last stage can hold rows past qend (their loads repeat row
    // qend - 1): once its loads have landed, their lse becomes +inf, so that
    // their P and dS are exactly zero and no stage needs a per-row mask.
    auto seal = [&](int u, int q0) __attribute__((always_inline)) {
        const int rows = qend - q0;
        if (rows < BQ) {
            if (tid >= rows && tid < BQ) ((lds_f32*)(L + VEC + u * 256))[tid] = __builtin_inff();
            __syncthreads();
        }
    };
    wait_lds_dma();
    __syncthreads();
    for (int ts = 0; ts < n_st; ts += 2) {
        const int q0 = qbeg + ts * BQ;
        if (ts + 1 < n_st) issue(q0 + BQ, 1);
        seal(0, q0);
        if (busy) compute(std::integral_constant<int, 0>{}, q0);
        wait_lds_dma();
        __syncthreads();
        if (ts + 1 >= n_st) break;
        if (ts + 2 < n_st) issue(q0 + 2 * BQ, 0);
        seal(1, q0 + BQ);
        if (busy) compute(std::integral_constant<int, 1>{}, q0 + BQ);
        wait_lds_dma();
        __syncthreads();
    }

    // (every wave is past the last stage's barrier: the stage buffers are free)
    if (busy) {
        if (parts > 1) {
            float* const p = a.dkdv_part + (slot * NW + wave) * (2 * 32 * D);
            store_part<D>(p, dk, lane);
            store_part<D>(p + 32 * D, dv, lane);
        } else {
            lds_u8* const rows = L + wave * 32 * ROWB;
            const int ln = fresh_thread_index() & 63;
            store_rows<D>(rows, dk, a.scale, static_cast<__bf16*>(a.dk) + base + kw * st, st, k1 - kw, ln);
            asm volatile("" ::: "memory");
            store_rows<D>(rows, dv, 1.f, static_cast<__bf16*>(a.dv) + base + kw * st, st, k1 - kw, ln);
        }
    }
}

// Adds up the parts of split tiles, in order: one wave per 32 rows and 32
// dimensions of one tensor. Blocks [0, n_q) take the query tiles' dQ (where
// split), then the split key tiles' dK and dV.
template <int D>
__global__ __launch_bounds__(64) void bwd_sum_kernel(const BwdArgs a, int n_q) {
    constexpr int DB = D / 32, NW = 4, U = 4;
    const int lane = threadIdx.x, hw = lane >> 5, l32 = lane & 31;
    int i = blockIdx.x;
    const bool is_q = i < n_q;
    if (!is_q) i -= n_q;
    const int d = i % DB;
    i /= DB;
    const int tensor = is_q ? 0 : i % 2;
    if (!is_q) i /= 2;
    const int wave = i % NW;
    i /= NW;  // split tile
    const int BH = a.B * a.H;
    int bh, t, parts, chunk, r0, r1;
    const float* p;
    int64_t step;  // from part to part
    __bf16* out;
    if (is_q) {
        parts = a.q_parts;
        bh = i / a.q_tiles;
        t = i % a.q_tiles;
        tile_rows(a, t, kBwdQTile, a.q_ref_tiles, a.q_chunk_tiles, chunk, r0, r1);
        step = NW * 32 * D;
        p = a.dq_part + (static_cast<int64_t>(i) * parts * NW + wave) * (32 * D);
        out = static_cast<__bf16*>(a.dq);
    } else {
        const int ref = a.k_ref_parts > 1 ? a.k_ref_tiles * BH : 0;
        int64_t slot;
        if (i < ref) {
            parts = a.k_ref_parts;
            slot = static_cast<int64_t>(i) * parts;
            bh = i / a.k_ref_tiles;
            t = i % a.k_ref_tiles;
        } else {
            const int rest = a.k_tiles - a.k_ref_tiles;
            parts = a.k_chunk_parts;
            slot = static_cast<int64_t>(ref) * a.k_ref_parts + static_cast<int64_t>(i - ref) * parts;
            bh = (i - ref) / rest;
            t = a.k_ref_tiles + (i - ref) % rest;
        }
        tile_rows(a, t, kBwdKTile, a.k_ref_tiles, a.k_chunk_tiles, chunk, r0, r1);
        step = NW * 2 * 32 * D;
        p = a.dkdv_part + (slot * NW + wave) * (2 * 32 * D) + tensor * (32 * D);
        out = static_cast<__bf16*>(tensor == 0 ? a.dk : a.dv);
    }
    const int row = r0 + 32 * wave + l32;
    if (r0 + 32 * wave >= r1) return;
    p += 4 * d * 256 + 4 * lane;
    f32x4_t acc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = f32x4_t{};
    for (int j = 0; j < parts; j += U) {
        f32x4_t x[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                x[u][g] = *reinterpret_cast<const f32x4_t*>(p + min(j + u, parts - 1) * step + g * 256);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j + u < parts) {
#pragma unroll
                for (int g = 0; g < 4; ++g) acc[g] += x[u][g];
            }
    }
    if (row >= r1) return;
    const float sc = tensor == 0 ? a.scale : 1.f;
    out += ((static_cast<int64_t>(bh / a.H) * a.L + row) * a.H + bh % a.H) * D + 32 * d + 4 * hw;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        bf16x4_t w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(acc[g][e] * sc);
        *reinterpret_cast<bf16x4_t*>(out + 8 * g) = w;
    }
}

template <int D>
hipError_t launch_bwd(const BwdArgs& a, hipStream_t s) {
    const int64_t bh = static_cast<int64_t>(a.B) * a.H;
    const int64_t g0 = static_cast<int64_t>((a.L + 63) / 64) * bh;
    const int64_t g1 = a.q_tiles * bh * a.q_parts;
    const int64_t rest = a.k_tiles - a.k_ref_tiles;
    const int64_t g2 = (a.k_ref_tiles * static_cast<int64_t>(a.k_ref_parts) + rest * a.k_chunk_parts) * bh;
    const int64_t n_q = a.q_parts > 1 ? a.q_tiles * bh * 4 * (D / 32) : 0;
    const int64_t n_k = ((a.k_ref_parts > 1 ? a.k_ref_tiles : 0) + (a.k_chunk_parts > 1 ? rest : 0)) * bh * 4 * 2 * (D / 32);
    if (g0 > INT32_MAX || g1 > INT32_MAX || g2 > INT32_MAX || n_q + n_k > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(bwd_delta_kernel<D>, dim3(static_cast<unsigned>(g0)), dim3(256), 0, s,
                       static_cast<const __bf16*>(a.o), static_cast<const __bf16*>(a.dout), a.delta,
                       a.B, a.L, a.H);
    hipLaunchKernelGGL(bwd_dq_kernel<D>, dim3(static_cast<unsigned>(g1)), dim3(kDqThreads), 0, s, a);
    hipLaunchKernelGGL(bwd_dkdv_kernel<D>, dim3(static_cast<unsigned>(g2)), dim3(kDkdvThreads), 0, s, a);
    if (n_q + n_k > 0)
        hipLaunchKernelGGL(bwd_sum_kernel<D>, dim3(static_cast<unsigned>(n_q + n_k)), dim3(64), 0, s, a,
                           static_cast<int>(n_q));
    return hipGetLastError();
}

// Workspace of the allocation-free backward entry point: delta for up to
// kBwdScratchFloats (batch, head, token) rows, in a device-global array that
// every GPU the library runs on holds until the process ends. Host code never
// passes this symbol to a kernel (on the host it names a stand-in, not the
// device copy): it uses the address hipGetSymbolAddress returns for the
// current device.
__device__ __align__(256) float scratch[kBwdScratchFloats];

constexpr int kMaxScratchDevices = 64;

}  // namespace

hipError_t launch_attn_bwd_bf16(const BwdArgs& a, int head_dim, hipStream_t s) {
    if (head_dim == 128) return launch_bwd<128>(a, s);
    if (head_dim == 64) return launch_bwd<64>(a, s);
    return hipErrorInvalidValue;
}

hipError_t bwd_scratch_address(float** out) {
    // One address per device, looked up once, with that device current
    // (every GPU holds its own copy of the array).
    static std::atomic<float*> addr[kMaxScratchDevices];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
    float* p = addr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        void* q = nullptr;
        e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (q == nullptr) return hipErrorInvalidSymbol;
        p = static_cast<float*>(q);
        addr[dev].store(p, std::memory_order_release);  // concurrent first calls store the same value
    }
    *out = p;
    return hipSuccess;
}

}  // namespace tmk
