// Sparse causal attention forward for gfx950 (MI355X, CDNA4).
//
// Computes, for every query row i of chunk a, O_i = softmax_j(scale * q_i.k_j) v_j
// over the keys j of {c_0, c_{a-W}, ..., c_a} (TalkingMachines, Sec. 4.2: the
// sparse attention pattern and its attention equation). The key set of a query
// chunk is a union of at most a few contiguous key ranges; query tiles never
// straddle a chunk, so every row of a tile shares its ranges, key tiles are
// visited only inside those ranges (masked blocks are never loaded), and only
// the last key tile of a range needs a column mask.
//
// bf16 kernel: one workgroup of 8 waves (two per SIMD) per 256-row query tile,
// 32 query rows per wave; all 8 waves share each K/V tile staged in LDS.
// Per 64-key tile the work is
//   S^T (keys x queries) = K Q^T with v_mfma_f32_32x32x16_bf16, K from LDS,
//     Q^T held in registers for the whole loop;
//   the softmax in fp32 on the MFMA output layout (each lane owns one query
//     column and half of its keys): x = S*scale*log2(e) - m against a lazily
//     raised running max m, P = exp2(x), rounded to bf16 for the P V product,
//     row sums of P in fp32;
//   O^T (head_dim x queries) += V^T P^T with the same MFMA, P^T straight from
//     registers. From the KV cache, whose V blocks are stored dimension-major,
//     the V tile lands in LDS as V^T and each operand is one 16-byte read; the
//     K rows are fed to the S MFMA in a permuted order that makes each lane's
//     P^T elements 8 consecutive keys. From row-major V (whole-sequence calls
//     on caller tensors) the operand is read with the gfx950 transposing read.
// The loop is software-pipelined so that every wave keeps the matrix core fed
// with its own VALU work in between (a wave's VALU work overlaps the MFMAs of
// the same wave far better than those of the other wave on its SIMD): while
// the MFMAs of S(t+1) run, the same wave forms P(t); while those of P(t) V(t)
// run, it scales S(t+1). Each MFMA is preceded by the LDS read of the operand
// fragment four MFMAs ahead. K/V tiles stream through four LDS buffers per
// tensor, filled by direct global->LDS loads two (V) and four (K) tiles ahead,
// with one barrier per tile.
//
// Query tiles that do not fill the GPU share their keys out in parts, each with
// a running max of its own: over several workgroups, merged by a second kernel,
// where the call has a workspace; else in turn in one workgroup, which merges
// them itself. The arithmetic is the same, and so are the bits.
//
// fp32 kernel: fp32 MFMAs (v_mfma_f32_32x32x2_f32) with an exact running max,
// operands loaded from global memory by the lanes that feed them; the keys of a
// query tile may be shared out over a workgroup's waves.

#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "tm_device.h"
#include "tm_internal.h"

namespace tmk {
namespace {

typedef __attribute__((address_space(3))) bf16x4_t lds_bf16x4_t;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;
typedef __attribute__((address_space(3))) f32x4_t lds_f32x4_t;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(5))) f32x4_t lane_f32x4_t;  // private memory of a lane

// Threads per workgroup of the bf16 kernel: 8 waves (two per SIMD) sharing
// every K/V tile staged in LDS.
constexpr int kBf16Threads = 512;
constexpr int kMaxLds = 160 * 1024;  // of a workgroup
// Wait until at most N LDS operations (and scalar loads) of this wave are
// outstanding; vector-memory and export counts are left unconstrained.
template <int N>
__device__ __forceinline__ void wait_lds_reads() {
    static_assert(N >= 0 && N < 16, "lgkmcnt field");
    __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// The same, except that the newest N direct loads may still be in flight
// (vector-memory operations complete in issue order for this count).
template <int N>
__device__ __forceinline__ void wait_lds_dma_but() {
    static_assert(N >= 0 && N < 16, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0 | N);
}

// Keeps x in a register at this point of the program: the empty statement
// takes x as input and output, so the computation of x cannot be moved past
// it (the compiler would otherwise sink work that is only used after a branch
// or a barrier, away from the MFMAs it is meant to overlap).
__device__ __forceinline__ float pin(float x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Query rows [q0, q1) of tile `tile` and its key ranges. Mode 0 takes the
// ranges from the kernel arguments; mode 1 derives them from the geometry.
struct TileRanges {
    int q0, q1;
    int n;         // number of ranges
    int b0, e0;    // the first two ranges (a whole sequence has no more)
    int b1, e1;
};

// Rows [q0, q1) of tile `idx` among the `nt` tiles that cover the rows
// [begin, end) of one chunk: the chunk's 32-row blocks are split as evenly as
// possible, the first tiles one block larger where they do not divide evenly,
// so tiles take about equally long; only the chunk's last block may be
// partial. With nt = ceil((end - begin) / BM) a tile has at most BM / 32 blocks.
__device__ __forceinline__ void split_rows(int begin, int end, int nt, int idx, int& q0, int& q1) {
    const int blocks = (end - begin + 31) / 32;
    const int each = blocks / nt, more = blocks - each * nt;
    q0 = begin + 32 * (idx * each + min(idx, more));
    q1 = min(begin + 32 * ((idx + 1) * each + min(idx + 1, more)), end);
}

__device__ __forceinline__ TileRanges plan_tile(const AttnArgs& a, int tile, int BM) {
    TileRanges t;
    if (a.mode == 0) {
        split_rows(0, a.Lq, a.n_qtiles, tile, t.q0, t.q1);
        t.n = a.n_ranges;
        t.b0 = a.range_begin[0];
        t.e0 = a.range_end[0];
        t.b1 = a.range_begin[1];
        t.e1 = a.range_end[1];
        return t;
    }
    // Mode 1: tiles are ordered heaviest first (the last chunks see the most
    // keys), so walk the natural order backwards.
    const int nat = a.n_qtiles - 1 - tile;
    int chunk;
    if (nat < a.ref_tiles) {
        chunk = 0;
        split_rows(0, a.ref_tok, a.ref_tiles, nat, t.q0, t.q1);
    } else {
        const int u = nat - a.ref_tiles;
        const int before = u / a.chunk_tiles;
        chunk = 1 + before;
        const int cs = a.ref_tok + (chunk - 1) * a.chunk_tok;
        const int ce = min(cs + a.chunk_tok, a.seq_len);
        split_rows(cs, ce, (ce - cs + BM - 1) / BM, u - before * a.chunk_tiles, t.q0, t.q1);
    }
    t.n = 1;
    t.b0 = t.b1 = t.e1 = 0;
    t.e0 = a.ref_tok;
    if (chunk > 0) {
        const int lo = max(1, chunk - a.window);
        const int end = min(a.ref_tok + chunk * a.chunk_tok, a.seq_len);
        if (lo == 1) {  // c_0 and c_1 are adjacent: one range
            t.e0 = end;
        } else {
            t.n = 2;
            t.b1 = a.ref_tok + (lo - 1) * a.chunk_tok;
            t.e1 = end;
        }
    }
    return t;
}

// 64-key tiles of a query tile's ranges.
__device__ __forceinline__ int key_tiles(const AttnArgs& a, const TileRanges& t) {
    if (a.mode == 0) return a.n_ktiles;
    return (t.e0 - t.b0 + kKeyTile - 1) / kKeyTile + (t.n > 1 ? (t.e1 - t.b1 + kKeyTile - 1) / kKeyTile : 0);
}

// Range r of a tile. A cache call (CACHE) may have up to kMaxRanges, in the
// kernel arguments; a whole sequence has at most two, held in registers.
template <bool CACHE>
__device__ __forceinline__ int range_begin(const AttnArgs& a, const TileRanges& t, int r) {
    return CACHE ? a.range_begin[r] : (r == 0 ? t.b0 : t.b1);
}
template <bool CACHE>
__device__ __forceinline__ int range_end(const AttnArgs& a, const TileRanges& t, int r) {
    return CACHE ? a.range_end[r] : (r == 0 ? t.e0 : t.e1);
}

__device__ __forceinline__ f32x16_t mfma32x32x16(bf16x8_t a, bf16x8_t b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// ----------------------------------------------------------------------------
// bf16 MFMA kernel
// ----------------------------------------------------------------------------
// LDS holds four K tiles and four V tiles, each BN rows of D bf16 with no
// padding. Every 16-byte chunk of a row sits at chunk position
// (chunk ^ swz(row)), which spreads both the K operand reads (same chunk of
// consecutive rows) and the transposing V reads (two adjacent chunks of four
// consecutive rows) over distinct banks. Tiles are filled by direct
// global->LDS loads (global_load_lds_dwordx4): each wave instruction writes
// 1 KB of LDS linearly, so each lane fetches the global chunk that belongs at
// its LDS position (lds_swizzle).

// V^T tile: D rows of 64 keys (128 bytes, 8 chunks of 8 keys). Chunk c of row
// d sits at position c ^ vt_swizzle(d): over any 16 consecutive rows the pair
// (row parity, position) takes all 16 values, so 16 lanes reading the same
// chunk of 16 consecutive rows hit 64 distinct banks.
__device__ __forceinline__ int vt_swizzle(int d) { return (d >> 1) & 7; }




// The merge of a row's parts, added in order: the running max m (log2 domain)
// and row sum l of the parts so far, and the factors of their O and of the next
// part's. A part whose row sum is zero (only scores of -inf) adds nothing. Every
// rounding is spelled out: both places that merge give the same bits.
struct RowMerge {
    float m = kNegInf, l = 0.f;
    float keep = 0.f, take = 0.f;
    __device__ __forceinline__ void next(float mi, float li) {
        const float mx = li != 0.f ? fmaxf(m, mi) : m;
        keep = l != 0.f ? __builtin_amdgcn_exp2f(m - mx) : 0.f;
        take = li != 0.f ? __builtin_amdgcn_exp2f(mi - mx) : 0.f;
        l = fmaf(take, li, __fmul_rn(l, keep));
        m = mx;
    }
    __device__ __forceinline__ float fold(float o, float oi) const { return fmaf(take, oi, __fmul_rn(o, keep)); }
};

// A workgroup takes a query tile or a part of a split one. TURN > 0 (a call
// without a workspace): TURN workgroups take a split tile, a share of its rows
// and all of its parts in turn each. Bound by a wave's own chain: with one busy
// wave on a SIMD a key tile takes 0.8 us and not 1.1, and the parts' ends, in a
// branch of the one continuous walk, hardly show. 480p chunk with 1, 3, 5 heads
// (13, 4, 2 parts): 143, 144, 148 us; 44, 85, 130 with a workspace; 187, 190, 191
// unsplit; 735, 361, 279 with a walk of its own per part.
template <int D, bool VT, bool OF32, int TURN>
__global__ __launch_bounds__(kBf16Threads, 1) void attn_fwd_bf16_kernel(const AttnArgs a) {
    constexpr int BM = kTileRowsBf16;  // query rows per workgroup
    constexpr int BN = kKeyTile;       // keys per tile
    constexpr int CPR = D / 8;         // 16-byte chunks per key row
    constexpr int ROWB = D * 2;        // bytes per key row
    constexpr int TILEB = BN * ROWB;
    constexpr int NW = kBf16Threads / 64;            // waves per workgroup, 32 query rows each
    constexpr int NI = TILEB / (kBf16Threads * 16);  // direct loads per thread per tensor per tile
    constexpr int KK = D / 16;  // MFMA k-steps over head_dim
    constexpr int DB = D / 32;  // 32-row blocks of O^T
    constexpr int NK = 2 * KK;  // K fragments per tile = score MFMAs per wave
    constexpr int NV = 4 * DB;  // V fragments per tile = P.V MFMAs per wave
    constexpr int NF = NK + NV;
    constexpr int RING = 4;        // fragments read ahead of their MFMA
    constexpr int EPG = 32 / NK;   // P elements formed per score MFMA
    constexpr int FPG = 32 / NV;   // scores scaled per P.V MFMA
    constexpr int NBUF = 4;        // LDS buffers per tensor (a power of two)
    static_assert(NI * kBf16Threads * 16 == TILEB, "tile must split evenly over the threads");
    static_assert(BM == NW * 32, "one 32-row query block per wave");
    static_assert(NF % RING == 0 && NK >= RING && EPG % 2 == 0, "fragment ring layout");

    // K tile j sits in buffer j % 4 of the first four, V tile j in buffer
    // j % 4 of the last four; behind them, where there is room, O of the parts
    // before (TURN).
    constexpr int SUMB = TURN > 0 ? NW / TURN * 32 * D * 4 : 0;
    constexpr bool LSUM = SUMB > 0 && 2 * NBUF * TILEB + SUMB <= kMaxLds;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * NBUF * TILEB + (LSUM ? SUMB : 0)];
    lds_u8* const L = (lds_u8*)(smem);
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(L));

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int hw = lane >> 5;   // half-wave: which 8-element k-slice a lane feeds
    const int l32 = lane & 31;  // the query column (and operand row) a lane owns

    // Whole tiles first, then the parts of the split ones (n_whole is a
    // multiple of the XCDs), a tile's parts next to each other.
    const int total = a.n_qtiles * a.B * a.H;
    const bool split = static_cast<int>(blockIdx.x) >= a.n_whole;
    int id, part = 0;
    if (!split) {
        id = xcd_logical_id(blockIdx.x, a.n_whole);
    } else {
        const int each = TURN > 0 ? TURN : a.parts;  // workgroups per split tile
        const int sid = xcd_logical_id(blockIdx.x - a.n_whole, (total - a.n_whole) * each);
        id = a.n_whole + sid / each;
        part = sid % each;
    }
    const int tile = id % a.n_qtiles;
    const int bh = id / a.n_qtiles;
    const int head = bh % a.H;
    const int bat = bh / a.H;
    TileRanges tr = plan_tile(a, tile, BM);
    if constexpr (TURN > 0) {
        if (split) {
            tr.q0 += part * (BM / TURN);
            tr.q1 = min(tr.q1, tr.q0 + BM / TURN);
            if (tr.q0 >= tr.q1) return;
            part = 0;
        }
    }

    const __bf16* qp = static_cast<const __bf16*>(a.q) + bat * a.q_sb + head * a.q_sh;
    const __bf16* kp = static_cast<const __bf16*>(a.k) + bat * a.k_sb + head * a.k_sh;
    const __bf16* vp = static_cast<const __bf16*>(a.v) + bat * a.v_sb + head * a.v_sh;

    // ---- key tiles: the tiles of range 0, then those of range 1, ... A Walk
    // stands in range r: tile j of the walk starts at key kb + BN * j as long
    // as that lies below the range's end ke. Walks only move forward.
    struct KeyTile {
        int k0, ke;
    };
    struct Walk {
        int kb, ke, r;
    };
    int n = VT ? a.n_ktiles : key_tiles(a, tr);
    // Parts of the tile (no more than it has key tiles): part i takes tiles
    // [n i / parts, n (i + 1) / parts).
    int parts = 1;
    if (split) {
        parts = min(a.parts, n);
        if (part >= parts) return;
    }
    // one past the walk's last tile in the current range
    auto tiles_end = [](const Walk& w) { return (w.ke - w.kb + BN - 1) / BN; };
    // Tile j (clamped to the walk's last tile).
    auto tile_at = [&](Walk& w, int j) __attribute__((always_inline)) {
        int e = tiles_end(w);
        while (j >= e && w.r + 1 < tr.n) {
            ++w.r;
            w.kb = range_begin<VT>(a, tr, w.r) - BN * e;
            w.ke = range_end<VT>(a, tr, w.r);
            e = tiles_end(w);
        }
        return KeyTile{w.kb + BN * min(j, e - 1), w.ke};
    };

    // ---- direct global->LDS loads of one tile. Rows past the range end
    // re-read the range's last row (finite data; its scores are masked). A V^T
    // tile takes, for each dimension d, the 8-key groups of the tile from the
    // cache's V block(s); groups past the range end re-read the group holding
    // the range's last key (its other columns are the append's zeros). Each
    // wave loads NI blocks of 1 KB per tensor. The lane offsets from the
    // tile's scalar base are the same for every tile of a range except its
    // last, so they are planned again only for a range's last tile and for the
    // tile after it.
    auto plan = [&](uint32_t (&off)[NI], bool is_v, const KeyTile& t) __attribute__((always_inline)) {
        // the thread index read afresh: the per-lane terms below are then
        // recomputed on this rare path instead of being kept live (spilled)
        // across the key loop
        const int tix = fresh_thread_index();
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int ch = i * kBf16Threads + tix;
            if (!is_v || !VT) {
                const int row = min(ch / CPR, t.ke - 1 - t.k0);
                const int gc = (ch % CPR) ^ lds_swizzle<D>(ch / CPR);
                const int64_t st = is_v ? a.v_st : a.k_st;
                off[i] = static_cast<uint32_t>((row * st + gc * 8) * 2);
            } else {
                const int d = ch >> 3;
                const int b0 = t.k0 & ~63;  // first cache block of the tile
                const int g = min(t.k0 + 8 * ((ch & 7) ^ vt_swizzle(d)), (t.ke - 1) & ~7) - b0;
                off[i] = static_cast<uint32_t>(((g >> 6) * (64 * D) + d * 64 + (g & 63)) * 2);
            }
        }
    };
    const uint32_t lds_wave = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(wave * 1024));
    // Byte offsets of K buffer j % 4 from the start of LDS, and of V buffer
    // j % 4 from the start of the V buffers (NBUF * TILEB further on).
    auto kbuf = [](int j) { return static_cast<uint32_t>((j & (NBUF - 1)) * TILEB); };
    auto vbuf = [](int j) { return static_cast<uint32_t>((j & (NBUF - 1)) * TILEB); };
    auto kbase = [&](const KeyTile& t) { return uniform_ptr(kp + static_cast<int64_t>(t.k0) * a.k_st); };
    auto vbase = [&](const KeyTile& t) {
        return VT ? uniform_ptr(vp + static_cast<int64_t>(t.k0 & ~63) * D)
                  : uniform_ptr(vp + static_cast<int64_t>(t.k0) * a.v_st);
    };
    // Load i (0 <= i < NI) of two tiles issued together: source p0 + lane
    // offset o0 into LDS byte offset l0, and likewise p1, o1, l1.
    auto dma_pair = [&](int i, const void* p0, uint32_t o0, uint32_t l0, const void* p1, uint32_t o1,
                        uint32_t l1) __attribute__((always_inline)) {
        const uint32_t blk = lds_base + lds_wave + i * NW * 1024;
        lds_dma16x2(p0, o0, l0 + blk, p1, o1, l1 + blk);
    };

    // ---- per-lane LDS byte offsets of the operand fragments within a tile.
    // K fragment (kk, kb): row l32 + 32*kb (permuted with VT), chunk 2*kk + hw.
    const int k_row = VT ? k_perm(l32) : l32;
    const int k_swz = lds_swizzle<D>(k_row);
    uint32_t koff[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) koff[kk] = k_row * ROWB + (((2 * kk + hw) ^ k_swz) << 4);
    // V fragment (j, d): with VT, row 32*d + l32 of the V^T tile, keys
    // 16*j + 8*hw .. + 7; else two transposing reads of the row-major tile,
    // rows 16*j + 4*hw + gi/4 (and + 8), element columns 32*d + 16*(grp & 1) +
    // 4*(gi & 3).
    constexpr int kVtRowBytes = 64 * 2;  // a V^T row: 64 keys
    const int grp = lane >> 4, gi = lane & 15;
    const int v_row = 4 * hw + (gi >> 2);
    const int v_swz_lo = lds_swizzle<D>(v_row), v_swz_hi = lds_swizzle<D>(v_row + 8);
    const int v_cbase = 2 * (grp & 1) + ((gi & 3) >> 1);
    const int v_half = (gi & 1) * 8;
    uint32_t voff[VT ? 4 : 2 * DB];
    if constexpr (VT) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            voff[j] = NBUF * TILEB + l32 * kVtRowBytes + (((2 * j + hw) ^ vt_swizzle(l32)) << 4);
    } else {
#pragma unroll
        for (int d = 0; d < DB; ++d) {
            const int cc = 4 * d + v_cbase;
            voff[2 * d] = NBUF * TILEB + v_row * ROWB + ((cc ^ v_swz_lo) << 4) + v_half;
            voff[2 * d + 1] = NBUF * TILEB + (v_row + 8) * ROWB + ((cc ^ v_swz_hi) << 4) + v_half;
        }
    }
    // Fragment s of a tile's stream: K fragments 0..NK-1 (kk = s/2, kb = s%2)
    // from the K buffer at byte offset kb_off, then V fragments
    // (j = (s-NK)/DB, d = (s-NK)%DB) from the V buffer at vb_off. Lane offset
    // plus a constant: the buffer offsets fold into the read's immediate.
    auto read_frag = [&](int s, uint32_t kb_off, uint32_t vb_off) __attribute__((always_inline)) {
        bf16x8_t f;
        if (s < NK) {
            const int kk = s >> 1, kb = s & 1;
            f = *reinterpret_cast<const lds_bf16x8_t*>(L + koff[kk] + (kb_off + kb * 32 * ROWB));
        } else {
            const int j = (s - NK) / DB, d = (s - NK) % DB;
            if constexpr (VT) {
                f = *reinterpret_cast<const lds_bf16x8_t*>(L + voff[j] + (vb_off + d * 32 * kVtRowBytes));
            } else {
                const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (lds_bf16x4_t*)(L + voff[2 * d] + (vb_off + 16 * j * ROWB)));
                const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (lds_bf16x4_t*)(L + voff[2 * d + 1] + (vb_off + 16 * j * ROWB)));
                f = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
        return f;
    };

    // ---- state
    f32x16_t acc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i) acc[i] = f32x16_t{};
    float m_run;            // running max in the scaled log2 domain (lazy)
    // Lanes whose row has had no finite score yet. Their running max is 0, so that
    // scores of -inf add nothing; the first tile that has a finite score sets it to
    // its own maximum, which may be far below.
    uint64_t fresh = 0;
    float l_run = 0.f;      // this lane's partial row sum
    const float c = a.scale_log2;
    // S^T output layout: register i of block kb holds key 32*kb + (VT ?
    // 16*(i/8) + 8*hw + i%8 : 8*(i/4) + 4*hw + i%4) of the tile, query l32.
    auto key_of = [&](int kb, int i) {
        return 32 * kb + (VT ? 16 * (i / 8) + 8 * hw + (i % 8) : 8 * (i / 4) + 4 * hw + (i % 4));
    };
    auto mask_tile = [&](f32x16_t (&s)[2], const KeyTile& kt) __attribute__((always_inline)) {
        if (kt.k0 + BN > kt.ke) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (kt.k0 + key_of(kb, i) >= kt.ke) s[kb][i] = kNegInf;
        }
    };
    // Largest score of this query in the tile (both half-waves).
    auto row_max = [&](const f32x16_t (&s)[2]) __attribute__((always_inline)) {
        float mx = fmaxf(s[0][0], s[1][0]);
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, fmaxf(s[0][i], s[1][i]));
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
    };
    // P = exp2(x) for elements [e, e + 2) of x, rounded to bf16 into its P^T
    // operand slot (k-step e/8, slot e%8); the fp32 values are summed into *lt.
    // (Summing the rounded pair with v_dot2_f32_bf16 instead costs more: that
    // instruction waits for the MFMA in flight, a plain fp32 add does not.)
    auto form_p2 = [&](const f32x16_t (&x)[2], bf16x8_t (&pf)[4], int e, float& lt) __attribute__((always_inline)) {
        const float p0 = __builtin_amdgcn_exp2f(x[e >> 4][e & 15]);
        const float p1 = __builtin_amdgcn_exp2f(x[(e + 1) >> 4][(e + 1) & 15]);
        pf[e >> 3][e & 7] = static_cast<__bf16>(p0);
        pf[e >> 3][(e & 7) + 1] = static_cast<__bf16>(p1);
        lt = e < 4 ? p0 + p1 : lt + (p0 + p1);
    };

    // ---- prologue: tiles 0..3 of K and 0..1 of V in flight, S(0) and its
    // exact maximum (the lazy running max starts from it), x(0) = S(0)*c - m.
    uint32_t offk[NI], offv[NI];  // lane offsets of the loads of the current K and V tiles
    Walk ws{range_begin<VT>(a, tr, 0), range_end<VT>(a, tr, 0), 0};  // tile t+1 (scores)
    if (TURN == 0 && split) {
        // A part takes tiles [j0, j1) of the walk, numbered from 0 here. Loads
        // past j1 fetch tiles that exist.
        const int j0 = n * part / parts, j1 = n * (part + 1) / parts;
        tile_at(ws, j0);
        ws.kb += BN * j0;
        n = j1 - j0;
    }
    const KeyTile first = tile_at(ws, 0);
    Walk wv = ws, wk = ws;  // tiles t+2 (V loads) and t+4 (K loads)
    {
        Walk w = ws;
        uint32_t o0[NI], o1[NI];
        plan(o0, false, first);
        plan(o1, true, first);
#pragma unroll
        for (int i = 0; i < NI; ++i)
            dma_pair(i, kbase(first), o0[i], kbuf(0), vbase(first), o1[i], NBUF * TILEB + vbuf(0));
        const KeyTile k1t = tile_at(w, 1);
        plan(o0, false, k1t);
        plan(o1, true, k1t);
#pragma unroll
        for (int i = 0; i < NI; ++i)
            dma_pair(i, kbase(k1t), o0[i], kbuf(1), vbase(k1t), o1[i], NBUF * TILEB + vbuf(1));
        const KeyTile k2t = tile_at(w, 2), k3t = tile_at(w, 3);
        plan(o0, false, k2t);
        plan(o1, false, k3t);
#pragma unroll
        for (int i = 0; i < NI; ++i) dma_pair(i, kbase(k2t), o0[i], kbuf(2), kbase(k3t), o1[i], kbuf(3));
    }
    // ---- Q^T operand (B of the score MFMA): lane holds q[row][16*kk + 8*hw .. +8].
    // Issued behind the direct loads, so that both latencies pass together; the
    // waits the compiler places for them can only wait for more than needed.
    const int qrow = tr.q0 + wave * 32 + l32;
    const bool row_ok = qrow < tr.q1;
    bf16x8_t qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        if (row_ok) {
            qf[kk] = *reinterpret_cast<const bf16x8_t*>(qp + qrow * a.q_st + kk * 16 + hw * 8);
        } else {
            qf[kk] = bf16x8_t{};
        }
    }
    wait_lds_dma();
    __syncthreads();

    // A wave whose 32 query rows all lie past the tile's end (the last query
    // tile of a chunk) takes part in the loads and barriers only.
    const bool busy = __builtin_amdgcn_readfirstlane(static_cast<int>(tr.q0 + wave * 32 < tr.q1)) != 0;
    f32x16_t xa[2], xb[2];  // x(t) and S(t+1) / x(t+1), alternating roles
    m_run = 0.f;
    if (busy) {
        bf16x8_t kf[NK];
#pragma unroll
        for (int s = 0; s < NK; ++s) kf[s] = read_frag(s, kbuf(0), vbuf(0));
        xa[0] = xa[1] = f32x16_t{};
#pragma unroll
        for (int s = 0; s < NK; ++s) xa[s & 1] = mfma32x32x16(kf[s], qf[s >> 1], xa[s & 1]);
        mask_tile(xa, first);
        const float mx = row_max(xa);
        m_run = mx == kNegInf ? 0.f : mx * c;
        fresh = __ballot(mx == kNegInf);
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int i = 0; i < 16; ++i) xa[kb][i] = fmaf(xa[kb][i], c, -m_run);
    }
    bf16x8_t fr[RING];
#pragma unroll
    for (int s = 0; s < RING; ++s) fr[s] = read_frag(s, kbuf(1), vbuf(1));
    // Iteration 0 loads K(4) into the buffer of K(0), and a wave without rows
    // reaches that load at once: every wave must be done reading K(0) first.
    __syncthreads();

    // ---- main loop: iteration t, with x = x(t) and nx receiving S(t+1).
    // Stage 1: the score MFMAs of tile t+1, each with its share of P(t)
    // (exp2, bf16, row sum). Check: if some lane's row sum of the tile
    // exceeds 2^16 (a score more than 16 above the running max in the log2
    // domain, or a non-finite value), or has had no finite score yet, raise the
    // max to the tile's maximum (from none: set it), rescale O and the row sum,
    // and form P(t) again. Stage 2: the P.V MFMAs
    // of tile t, each with its share of x(t+1) = S(t+1)*c - m. Every MFMA is
    // preceded by the LDS read of the fragment RING MFMAs ahead; tile t+4 of
    // K and tile t+2 of V are loaded during stage 2. At the end each wave
    // waits for its loads of the previous iteration and the barrier publishes
    // K(t+2), K(t+3) and V(t+1).
    //
    // Tiles t+1 (scores), t+2 (V load) and t+4 (K load) move one tile on in
    // their range unless a tile among t+1..t+4 ends a range; only then (at
    // most a few iterations per range, and at the end of the walk) do their
    // walks move on, are the load offsets planned again and the mask of tile
    // t+1 decided.
    int event = 0;                 // smallest range-ending tile index >= the last refresh's t + 2
    const void* kptr = nullptr;    // K source of tile t+4
    const void* vptr = nullptr;    // V source of tile t+2
    bool mask_next = false;
    const int64_t kstep = static_cast<int64_t>(BN) * a.k_st * 2;  // bytes per tile of keys
    const int64_t vstep = static_cast<int64_t>(BN) * (VT ? D : a.v_st) * 2;
    auto refresh = [&](int t) __attribute__((always_inline)) {
        kptr = static_cast<const char*>(kptr) + kstep;
        vptr = static_cast<const char*>(vptr) + vstep;
        mask_next = false;
        // No else branch: with one, the compiler kept two copies of the state
        // and moved it on every iteration (12 of a tile's 260 instructions;
        // 480p chunk 888 -> 871 us).
        if (__builtin_expect(t + 4 >= event, 0)) {
            const KeyTile k4 = tile_at(wk, t + 4), v2 = tile_at(wv, t + 2), s1 = tile_at(ws, t + 1);
            mask_next = s1.k0 + BN > s1.ke;
            plan(offk, false, k4);
            plan(offv, true, v2);
            kptr = kbase(k4);
            vptr = vbase(v2);
            event = __builtin_amdgcn_readfirstlane(tiles_end(wv) - 1);
            // The range bounds may come from scalar loads, which share a
            // counter with the LDS reads and complete out of order: wait for
            // them here, on this rare path, so that no full wait lands on the
            // common path where fragment reads are still in flight.
            wait_lds_reads<0>();
        }
    };
    // TURN: where the current part ends, and the parts before it: O in LDS, or
    // where that is full in the lane's private memory (the registers are full too).
    // The walk goes on over a part's end; only the running max, the sum and O start
    // anew.
    int part_end = n / parts;
    RowMerge sum;
    lds_u8* const sum_l = L + 2 * NBUF * TILEB + __builtin_amdgcn_readfirstlane(wave) * (32 * D * 4) + lane * 16;
    lane_f32x4_t* sum_p = nullptr;
    f32x4_t sum_mem[TURN > 0 && !LSUM ? 4 * DB : 1];
    if constexpr (TURN > 0 && !LSUM) {
        sum_p = (lane_f32x4_t*)sum_mem;
        asm volatile("" : "+s"(sum_p));  // (else the compiler takes registers and spills in the key loop)
    }
    auto fold_part = [&]() __attribute__((always_inline)) {
        sum.next(m_run, l_run + __shfl_xor(l_run, 32));
        if (part == 0) {
#pragma unroll
            for (int i = 0; i < 16 * DB; ++i) acc[i / 16][i % 16] = sum.fold(0.f, acc[i / 16][i % 16]);
        } else {
#pragma unroll
            for (int d = 0; d < DB; ++d) {
                f32x4_t o[4];
#pragma unroll
                for (int g = 0; g < 4; ++g) o[g] = LSUM ? *(const lds_f32x4_t*)(sum_l + (4 * d + g) * 1024) : sum_p[4 * d + g];
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[d][i] = sum.fold(o[i / 4][i % 4], acc[d][i]);
            }
        }
    };
    // The barrier orders only this workgroup's LDS use: the compiler may not
    // move LDS accesses across it, and no wait is needed for the fragment
    // reads still in flight (their buffer is not written next).
    auto end_tile = [&]() __attribute__((always_inline)) {
        wait_lds_dma_but<2 * NI>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto iteration = [&](int u, int t, f32x16_t (&x)[2], f32x16_t (&nx)[2]) __attribute__((always_inline)) {
        const uint32_t kb1 = kbuf(u + 1), kb2 = kbuf(u + 2), vb0 = vbuf(u);
        refresh(t);
        bf16x8_t pf[4];
        float lt0, lt1;
        nx[0] = nx[1] = f32x16_t{};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < NK; ++g) {
            nx[g & 1] = mfma32x32x16(fr[g % RING], qf[g >> 1], nx[g & 1]);
            fr[g % RING] = read_frag(g + RING, kb1, vb0);
#pragma unroll
            for (int e = EPG * g; e < EPG * (g + 1); e += 2) form_p2(x, pf, e, (e & 2) ? lt1 : lt0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (__builtin_expect((__ballot(!(lt0 + lt1 <= 0x1p16f)) | fresh) != 0, 0)) {
            const float mx = row_max(x);
            const bool first = __builtin_amdgcn_inverse_ballot_w64(fresh) && mx != kNegInf;
            const float dm = first ? mx : fmaxf(mx, 0.f);
            const float alpha = first ? 1.f : __builtin_amdgcn_exp2f(-dm);  // (sum and O are still 0)
            fresh &= __ballot(mx == kNegInf);
            m_run += dm;
            l_run *= alpha;
#pragma unroll
            for (int d = 0; d < DB; ++d) acc[d] *= alpha;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 16; ++i) x[kb][i] -= dm;
#pragma unroll
            for (int e = 0; e < 32; e += 2) form_p2(x, pf, e, (e & 2) ? lt1 : lt0);
        }
        l_run += lt0 + lt1;
        if (mask_next) mask_tile(nx, tile_at(ws, t + 1));
        float nm = -m_run;
        const bool turn = TURN > 0 && t + 1 == part_end && t + 1 < n;
        if (turn) {  // tile t+1 starts a part: its exact maximum, as in the prologue
            const float mx = row_max(nx);
            nm = mx == kNegInf ? 0.f : -(mx * c);
            fresh = __ballot(mx == kNegInf);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            acc[k % DB] = mfma32x32x16(fr[(NK + k) % RING], pf[k / DB], acc[k % DB]);
            fr[(NK + k) % RING] = read_frag((NK + k + RING) % NF, NK + k + RING < NF ? kb1 : kb2, vb0);
#pragma unroll
            for (int e = FPG * k; e < FPG * (k + 1); ++e) nx[e >> 4][e & 15] = pin(fmaf(nx[e >> 4][e & 15], c, nm));
            if (k % (NV / NI) == NV / (2 * NI)) {
                const int i = k / (NV / NI);
                dma_pair(i, kptr, offk[i], kbuf(u), vptr, offv[i], NBUF * TILEB + vbuf(u + 2));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (TURN > 0) if (turn) {
            fold_part();
#pragma unroll
            for (int d = 0; d < DB; ++d) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4_t w{acc[d][4 * g], acc[d][4 * g + 1], acc[d][4 * g + 2], acc[d][4 * g + 3]};
                    if constexpr (LSUM) *(lds_f32x4_t*)(sum_l + (4 * d + g) * 1024) = w;
                    else sum_p[4 * d + g] = w;
                }
                acc[d] = f32x16_t{};
            }
            m_run = -nm;
            l_run = 0.f;
            ++part;
            part_end = n * (part + 1) / parts;
        }
        end_tile();
    };
    if (busy) {
        for (int t = 0; t < n; t += 4) {
            iteration(0, t, xa, xb);
            if (t + 1 >= n) break;
            iteration(1, t + 1, xb, xa);
            if (t + 2 >= n) break;
            iteration(2, t + 2, xa, xb);
            if (t + 3 >= n) break;
            iteration(3, t + 3, xb, xa);
        }
    } else {
        // the same loads and barriers, no arithmetic
        for (int t = 0; t < n; ++t) {
            refresh(t);
#pragma unroll
            for (int i = 0; i < NI; ++i)
                dma_pair(i, kptr, offk[i], kbuf(t), vptr, offv[i], NBUF * TILEB + vbuf(t + 2));
            end_tile();
        }
    }
    // no load may still be writing LDS; every wave is done with the tiles
    wait_lds_dma();
    __syncthreads();

    // ---- epilogue: normalise, store rows inside the tile, rounded to bf16
    // (nearest even) or, with OF32, as the fp32 values that rounding would take.
    // The rows go through the wave's share of the LDS (16-byte chunk c of row r
    // at c ^ (r & CM)), so that they are stored whole: in the MFMA layout a
    // store instruction would touch 32 rows for 16 or 32 bytes each (with the
    // queries behind the direct loads above, 3 us less per workgroup: one
    // 256-row tile over 20 key tiles 38.5 -> 35.7 us).
    float l_tot = l_run + __shfl_xor(l_run, 32);
    if constexpr (TURN > 0) {
        if (split) {
            fold_part();
            m_run = sum.m;
            l_tot = sum.l;
        }
    } else if (split) {
        // unnormalised, in registers' order: every store is a whole KB
        if (busy) {
            const int64_t at = (static_cast<int64_t>(id - a.n_whole) * a.parts + part) * NW + wave;
            float* const w = a.part + at * part_floats(D) + 4 * lane;
#pragma unroll
            for (int d = 0; d < DB; ++d)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<f32x4_t*>(w + (4 * d + g) * 256) =
                        f32x4_t{acc[d][4 * g], acc[d][4 * g + 1], acc[d][4 * g + 2], acc[d][4 * g + 3]};
            float* const ml = a.part + at * part_floats(D) + 32 * D;
            ml[lane] = m_run;
            ml[64 + lane] = l_tot;
        }
        return;
    }
    const float inv = 1.f / l_tot;
    {
        constexpr int ES = OF32 ? 4 : 2;       // bytes per element
        constexpr int OCPR = D * ES / 16;      // chunks per row
        constexpr int CM = OCPR < 16 ? 7 : 15;
        static_assert(NW * 32 * D * ES <= 2 * NBUF * TILEB, "output rows must fit the LDS");
        lds_u8* const rows = L + __builtin_amdgcn_readfirstlane(wave) * (32 * D * ES);
        const int ln = fresh_thread_index() & 63, row_l = ln & 31, half = ln >> 5;
        if (busy) {
#pragma unroll
            for (int d = 0; d < DB; ++d) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if constexpr (OF32) {
                        f32x4_t w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] = acc[d][4 * g + e] * inv;
                        *(lds_f32x4_t*)(rows + row_l * (D * ES) + (((8 * d + 2 * g + half) ^ (row_l & CM)) << 4)) = w;
                    } else {
                        bf16x4_t w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(acc[d][4 * g + e] * inv);
                        *(lds_bf16x4_t*)(rows + row_l * (D * ES) + (((4 * d + g) ^ (row_l & CM)) << 4) + 8 * half) = w;
                    }
                }
            }
            asm volatile("" ::: "memory");
            unsigned char* const op = static_cast<unsigned char*>(a.o) + (bat * a.o_sb + head * a.o_sh) * ES;
#pragma unroll
            for (int i = 0; i < 32 * OCPR / 64; ++i) {
                const int ch = 64 * i + ln, row = ch / OCPR;
                const f32x4_t w = *(const lds_f32x4_t*)(rows + row * (D * ES) + (((ch % OCPR) ^ (row & CM)) << 4));
                const int orow = tr.q0 + wave * 32 + row;
                if (orow < tr.q1)
                    *reinterpret_cast<f32x4_t*>(op + static_cast<int64_t>(orow) * a.o_st * ES + (ch % OCPR) * 16) = w;
            }
        }
    }
    if (row_ok) {
        if (a.lse != nullptr && hw == 0) {
            a.lse[(static_cast<int64_t>(bat) * a.H + head) * a.Lq + qrow] =
                (m_run + __log2f(l_tot)) * 0.69314718055994530942f;
        }
    }
}

// Merges the parts of the split query tiles: one wave per 32 query rows and 32
// output dimensions.
template <int D, bool OF32>
__global__ __launch_bounds__(64) void attn_merge_kernel(const AttnArgs a) {
    constexpr int BM = kTileRowsBf16, NW = BM / 32, DB = D / 32;
    const int lane = threadIdx.x, hw = lane >> 5, l32 = lane & 31;
    const int d = blockIdx.x % DB;
    const int wave = blockIdx.x / DB % NW;
    const int st = blockIdx.x / (DB * NW);  // split tile
    const int id = a.n_whole + st;
    const int tile = id % a.n_qtiles;
    const int bh = id / a.n_qtiles;
    const int head = bh % a.H;
    const int bat = bh / a.H;
    const TileRanges tr = plan_tile(a, tile, BM);
    if (tr.q0 + wave * 32 >= tr.q1) return;

    const float* p0 = a.part + (static_cast<int64_t>(st) * a.parts * NW + wave) * part_floats(D);
    constexpr int64_t step = NW * part_floats(D);  // from part to part
    // Four parts' loads in flight together, and the next four while these are
    // merged (the kernel is bound by their latency).
    constexpr int U = 4, G = kMaxParts / U;
    const int parts = min(a.parts, key_tiles(a, tr));
    float mi[2][U], li[2][U];
    f32x4_t ai[2][U][4];
    auto load = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float* p = p0 + min(U * i + u, parts - 1) * step;
            mi[i & 1][u] = p[32 * D + lane];
            li[i & 1][u] = p[32 * D + 64 + lane];
#pragma unroll
            for (int g = 0; g < 4; ++g)
                ai[i & 1][u][g] = *reinterpret_cast<const f32x4_t*>(p + (4 * d + g) * 256 + 4 * lane);
        }
    };
    RowMerge sum;
    f32x4_t acc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = f32x4_t{};
    load(0);
#pragma unroll
    for (int i = 0; i < G; ++i) {
        if (i + 1 < G && U * (i + 1) < parts) load(i + 1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (U * i + u < parts) {
                sum.next(mi[i & 1][u], li[i & 1][u]);
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[g][e] = sum.fold(acc[g][e], ai[i & 1][u][g][e]);
            }
        }
    }
    const float inv = 1.f / sum.l;
    const int qrow = tr.q0 + wave * 32 + l32;
    if (qrow >= tr.q1) return;
    const int64_t orow = bat * a.o_sb + head * a.o_sh + qrow * a.o_st + 32 * d + 4 * hw;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f32x4_t w = acc[g] * inv;
        if constexpr (OF32) {
            *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.o) + orow + 8 * g) = w;
        } else {
            bf16x4_t h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = static_cast<__bf16>(w[e]);
            *reinterpret_cast<bf16x4_t*>(static_cast<__bf16*>(a.o) + orow + 8 * g) = h;
        }
    }
    if (a.lse != nullptr && d == 0 && hw == 0)
        a.lse[(static_cast<int64_t>(bat) * a.H + head) * a.Lq + qrow] = (sum.m + __log2f(sum.l)) * 0.69314718055994530942f;
}

// ----------------------------------------------------------------------------
// fp32 MFMA kernel
// ----------------------------------------------------------------------------
// The same products with v_mfma_f32_32x32x2_f32 (fp32 operands and sums), one
// wave per 32 query rows and share of the keys. An fp32 MFMA takes 64 cycles
// for one register per operand, so operands need no LDS: the lanes load them
// from the cache hierarchy in the MFMA's layout (a lane's 16-byte load of a K
// row feeds four MFMAs), K of the next key block while the current one is
// computed. A workgroup's NW waves are split into a.key_groups groups of keys
// and NW / key_groups groups of 32 query rows; waves of one query group merge
// their (max, row sum, O) through LDS at the end, in a fixed order. Key groups
// fill the chip where query rows are few and also shorten the serial chain of
// a small call (a 32-key block takes about 1.7 us of one wave at D = 64); the
// host picks their number. Bound by the MFMAs plus what the operand loads cost
// (without any loads the loop is 1.3 times as fast): 2304 rows in 5 chunks, 8
// heads, D = 64: 66 us (76 TFLOP/s; 421 us as a VALU kernel with 4 lanes per
// row); 4000 rows, 48 heads, D = 128: 2.5 ms (86 TFLOP/s; 10.5 ms). V operands
// loaded one register at a time, not as 16-byte vectors, cost 20% more; masking
// every block and scaling scores apart from subtracting the maximum, 3-5%.
template <int D, int NW, bool VT>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) void attn_fwd_f32_kernel(const AttnArgs a) {
    constexpr int KC = D / 8;   // K chunks: 4 dimensions per half-wave
    constexpr int DB = D / 32;  // 32-row blocks of O^T
    constexpr int NR = 16 * DB; // O registers per lane
    __shared__ float part[NW / 2][NR + 2][64];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int hw = lane >> 5, l32 = lane & 31;
    const int kgs = a.key_groups;
    const int kg = wave % kgs, qg = wave / kgs;
    const int total = a.n_qtiles * a.B * a.H;
    const int id = xcd_logical_id(blockIdx.x, total);
    const int tile = id % a.n_qtiles;
    const int bh = id / a.n_qtiles;
    const int head = bh % a.H;
    const int bat = bh / a.H;
    const TileRanges tr = plan_tile(a, tile, 32 * (NW / kgs));

    const float* qp = static_cast<const float*>(a.q) + bat * a.q_sb + head * a.q_sh;
    const float* kp = static_cast<const float*>(a.k) + bat * a.k_sb + head * a.k_sh;
    const float* vp = static_cast<const float*>(a.v) + bat * a.v_sb + head * a.v_sh;
    const int qrow = tr.q0 + 32 * qg + l32;
    const bool row_ok = qrow < tr.q1;

    // Q^T operand: lane holds dimensions 8*kk + 4*hw .. + 3 of its query row.
    f32x4_t qf[KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
        qf[kk] = row_ok ? *reinterpret_cast<const f32x4_t*>(qp + qrow * a.q_st + 8 * kk + 4 * hw) : f32x4_t{};

    // This wave's share [jb, je) of the 32-key blocks of the tile's ranges.
    auto blocks_of = [&](int r) { return (range_end<VT>(a, tr, r) - range_begin<VT>(a, tr, r) + 31) / 32; };
    int n = 0;
    for (int r = 0; r < tr.n; ++r) n += blocks_of(r);
    const int jb = n * kg / kgs, je = n * (kg + 1) / kgs;
    const bool busy = jb < je && tr.q0 + 32 * qg < tr.q1;
    int r = 0, k0 = 0, ke = 0;  // current range, first key of the block, end of the range
    if (busy) {
        int j = jb;
        while (j >= blocks_of(r)) j -= blocks_of(r++);
        k0 = range_begin<VT>(a, tr, r) + 32 * j;
        ke = range_end<VT>(a, tr, r);
    }

    // K rows of the block at k0 (rows past the range end repeat its last row;
    // their scores are masked): lane's key k0 + l32, the Q operand's
    // dimensions. KR chunks are held, each reloaded once it is used.
    constexpr int KR = 8;
    f32x4_t kf[KR];
    auto load_k = [&](int kk, const float* row) __attribute__((always_inline)) {
        kf[kk % KR] = *reinterpret_cast<const f32x4_t*>(row + 8 * kk + 4 * hw);
    };
    auto k_base = [&](int first, int end) { return kp + static_cast<int64_t>(min(first + l32, end - 1)) * a.k_st; };
    // V^T operands of key group g of the block: v[d][e] feeds the MFMA of
    // score register 4*g + e (key 8*g + 4*hw + e of the block) into O block d,
    // zero past the range end. Row l32 of O block d is dimension 32*d + l32
    // with VT (a lane's 16-byte load holds 4 keys of one dimension), else
    // DB*l32 + d (a lane's load holds DB dimensions of one key).
    auto load_v = [&](float (&v)[DB][4], int g) __attribute__((always_inline)) {
        if constexpr (VT) {
            // from the first cache block of the tile (at most one block on)
            const int at = min(k0 + 8 * g + 4 * hw, (ke - 1) & ~3) - (k0 & ~63);
            const float* base = vp + static_cast<int64_t>(k0 >> 6) * (64 * D);
            const uint32_t off = (at >> 6) * (64 * D) + l32 * 64 + (at & 63);
#pragma unroll
            for (int d = 0; d < DB; ++d) {
                const f32x4_t w = *reinterpret_cast<const f32x4_t*>(base + off + d * 32 * 64);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[d][e] = w[e];
            }
        } else {
            typedef float vec_t __attribute__((ext_vector_type(DB)));
            // a wave-uniform row plus the lane's offset (0 or 4 rows on, which
            // fits 32 bits at the largest batch * heads)
            const bool full = k0 + 32 <= ke;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = k0 + 8 * g + e;
                const float* base = vp + static_cast<int64_t>(full ? row : min(row, ke - 1)) * a.v_st;
                const uint32_t rows = full ? 4 * hw : min(4 * hw, max(ke - 1 - row, 0));
                const vec_t w = *reinterpret_cast<const vec_t*>(base + (rows * static_cast<uint32_t>(a.v_st) + DB * l32));
#pragma unroll
                for (int d = 0; d < DB; ++d) v[d][e] = w[d];
            }
        }
        if (k0 + 32 > ke) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k0 + 8 * g + 4 * hw + e >= ke) {
#pragma unroll
                    for (int d = 0; d < DB; ++d) v[d][e] = 0.f;
                }
        }
    };

    f32x16_t acc[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d] = f32x16_t{};
    // Running max of the row (log2 domain), this lane's part of its sum. The max
    // starts from the lowest finite value, from which scores of -inf add nothing
    // (from -inf they would make the sum NaN).
    float m = -FLT_MAX, l = 0.f;
    const float c = a.scale_log2;
    if (busy) {
        const float* row = k_base(k0, ke);
#pragma unroll
        for (int kk = 0; kk < KR; ++kk) load_k(kk, row);
        for (int j = jb; j < je; ++j) {
            int nr = r, nk0 = k0 + 32, nke = ke;
            if (nk0 >= ke && j + 1 < je) {
                ++nr;
                nk0 = range_begin<VT>(a, tr, nr);
                nke = range_end<VT>(a, tr, nr);
            }
            const float* next = k_base(j + 1 < je ? nk0 : k0, nke);
            // V of the first VB key groups, in flight during the score MFMAs
            constexpr int VB = D == 64 ? 4 : 2;
            float v[VB][DB][4];
#pragma unroll
            for (int g = 0; g < VB; ++g) load_v(v[g], g);
            // S^T = K Q^T as two chains (half the additions in sequence)
            f32x16_t s0 = f32x16_t{}, s1 = f32x16_t{};
#pragma unroll
            for (int kk = 0; kk < KC; ++kk) {
                s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[kk % KR][0], qf[kk][0], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[kk % KR][1], qf[kk][1], s1, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[kk % KR][2], qf[kk][2], s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[kk % KR][3], qf[kk][3], s1, 0, 0, 0);
                if (kk + KR < KC) load_k(kk + KR, row);
                else load_k(kk + KR - KC, next);
            }
            row = next;
#pragma unroll
            for (int i = 0; i < 16; ++i) s0[i] += s1[i];
            if (k0 + 32 > ke) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (k0 + 8 * (i / 4) + 4 * hw + i % 4 >= ke) s0[i] = kNegInf;
            }
            float mx = s0[0];
#pragma unroll
            for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s0[i]);
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            const float m_new = fmaxf(m, fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * c);
            if (__any(m_new > m)) {
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                l *= alpha;
#pragma unroll
                for (int d = 0; d < DB; ++d) acc[d] *= alpha;
                m = m_new;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s0[i] = __builtin_amdgcn_exp2f(fmaf(s0[i], c, -m));
                l += s0[i];
            }
#pragma unroll
            for (int g = 0; g < 4; ++g) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int d = 0; d < DB; ++d)
                        acc[d] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[g % VB][d][e], s0[4 * g + e], acc[d], 0, 0, 0);
                if (g + VB < 4) load_v(v[g % VB], g + VB);
                __builtin_amdgcn_sched_barrier(0);  // no V loads further ahead (registers)
            }
            r = nr;
            k0 = nk0;
            ke = nke;
        }
    }
    l += __shfl_xor(l, 32);

    // Merge the key groups of a query group pairwise: the upper half of the
    // groups hand theirs over, the lower half fold them in.
    for (int half = kgs / 2; half >= 1; half /= 2) {
        float(*mine)[64] = part[qg * half + kg % half];
        if (kg >= half && kg < 2 * half) {
#pragma unroll
            for (int i = 0; i < NR; ++i) mine[i][lane] = acc[i / 16][i % 16];
            mine[NR][lane] = m;
            mine[NR + 1][lane] = l;
        }
        __syncthreads();
        if (kg < half) {
            const float m2 = mine[NR][lane];
            const float mm = fmaxf(m, m2);
            // (a group without keys, or whose scores are all -inf, has l = 0 and O = 0)
            const float f1 = exp2f(m - mm), f2 = exp2f(m2 - mm);
            l = l * f1 + mine[NR + 1][lane] * f2;
#pragma unroll
            for (int i = 0; i < NR; ++i) acc[i / 16][i % 16] = acc[i / 16][i % 16] * f1 + mine[i][lane] * f2;
            m = mm;
        }
        __syncthreads();
    }

    if (kg == 0 && row_ok) {
        float* op = static_cast<float*>(a.o) + bat * a.o_sb + head * a.o_sh + qrow * a.o_st;
        const float inv = 1.f / l;
        if constexpr (VT) {
#pragma unroll
            for (int d = 0; d < DB; ++d) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4_t w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = acc[d][4 * g + e] * inv;
                    *reinterpret_cast<f32x4_t*>(op + 32 * d + 8 * g + 4 * hw) = w;
                }
            }
        } else {
            typedef float vec_t __attribute__((ext_vector_type(DB)));
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                vec_t w;
#pragma unroll
                for (int d = 0; d < DB; ++d) w[d] = acc[d][i] * inv;
                *reinterpret_cast<vec_t*>(op + DB * (8 * (i / 4) + 4 * hw + i % 4)) = w;
            }
        }
        if (a.lse != nullptr && hw == 0) {
            a.lse[(static_cast<int64_t>(bat) * a.H + head) * a.Lq + qrow] =
                (m + log2f(l)) * 0.69314718055994530942f;
        }
    }
}

template <int D, bool VT, bool OF32>
void launch_bf16(const AttnArgs& a, hipStream_t s) {
    const int split = a.n_qtiles * a.B * a.H - a.n_whole;
    const dim3 block(kBf16Threads);
    if (split == 0 || a.part != nullptr) {
        hipLaunchKernelGGL((attn_fwd_bf16_kernel<D, VT, OF32, 0>), dim3(a.n_whole + split * a.parts), block, 0, s, a);
        if (split > 0)
            hipLaunchKernelGGL((attn_merge_kernel<D, OF32>), dim3(split * (kTileRowsBf16 / 32) * (D / 32)), dim3(64), 0, s,
                               a);
    } else if (4 * split <= kCUs) {
        // Four workgroups per split tile as long as all of them run at once: at
        // D = 128 the merged O fits their LDS, two need the lanes' private memory
        // (one head: 143 us with four, 186 with two).
        hipLaunchKernelGGL((attn_fwd_bf16_kernel<D, VT, OF32, 4>), dim3(a.n_whole + 4 * split), block, 0, s, a);
    } else {
        hipLaunchKernelGGL((attn_fwd_bf16_kernel<D, VT, OF32, 2>), dim3(a.n_whole + 2 * split), block, 0, s, a);
    }
}
template <int D, bool VT>
void launch_bf16_out(const AttnArgs& a, hipStream_t s) {
    if (a.o_f32) launch_bf16<D, VT, true>(a, s);
    else launch_bf16<D, VT, false>(a, s);
}

}  // namespace

hipError_t launch_attn_bf16(const AttnArgs& a, int head_dim, hipStream_t s) {
    if (head_dim == 128) {
        if (a.v_blocked) launch_bf16_out<128, true>(a, s);
        else launch_bf16_out<128, false>(a, s);
    } else if (head_dim == 64) {
        if (a.v_blocked) launch_bf16_out<64, true>(a, s);
        else launch_bf16_out<64, false>(a, s);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int D, int NW>
void launch_f32(const AttnArgs& a, hipStream_t s) {
    const dim3 grid(a.n_qtiles * a.B * a.H), block(NW * 64);
    if (a.v_blocked) hipLaunchKernelGGL((attn_fwd_f32_kernel<D, NW, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((attn_fwd_f32_kernel<D, NW, false>), grid, block, 0, s, a);
}

hipError_t launch_attn_f32(const AttnArgs& a, int head_dim, hipStream_t s) {
    if (head_dim == 128 && a.key_groups <= 4) launch_f32<128, 4>(a, s);
    else if (head_dim == 64 && a.key_groups <= 4) launch_f32<64, 4>(a, s);
    else if (head_dim == 64 && a.key_groups == 8) launch_f32<64, 8>(a, s);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace tmk
