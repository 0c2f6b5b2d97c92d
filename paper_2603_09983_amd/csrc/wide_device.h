// Expert FFN of batches of more than 32 tokens (Sec. 2.2 last line, experts as in App. D):
//      act = silu(W_gate x) * (W_up x)        (gate/up kernel)
//      o   = W_down act                       (down kernel)
//
// The small-batch kernels (stream.hip) keep an expert's B operand, all columns of up to 32 tokens, in the registers
// of sixteen wavefronts and stream whole weight rows past it.  With more tokens per expert, or with two token groups and
// rows of several panels, that operand has to come again for every tile.  Here an item is 64 weight rows (32 gate rows
// on 32 up rows, or 64 down rows) against 32 tokens of one expert's list; both operands pass through LDS in chunks of
// 512 columns, every load instruction one row's consecutive kilobyte, and the accumulators stay in registers for the
// whole contraction.  Bound: HBM for the weights (each is read from HBM once; an expert with more than 32 tokens reads
// its weights once per 32, the later times from the caches, as neighbouring items run at the same time).
//
// One workgroup of sixteen wavefronts per CU takes items b, b + G, .. and keeps three chunks in flight, across items
// (3 x 64 KB of weights).
//
// The order of the sums is the streaming kernels': wavefront w multiplies columns 32 w .. 32 w + 31 of every chunk, the
// chunks of a row in ascending order, and an item's sixteen partial results are added through LDS in wavefront order.  So a
// token's outputs have the same bits whichever of the kernels runs (contractions of up to kPanelMax columns), whatever else
// is in the batch and wherever the item lies in the list.  It costs an item's end two barriers and 128 KB of LDS traffic each
// way (64 rows; with 32 rows the partial results have LDS of their own).
//
// Rows of several panels (K > kPanelMax) start at a chunk that follows from the row: with rows of 8 KB and more all rows'
// kilobytes of one chunk lie in few of an L2's sixteen channels, and workgroups that start together would all be in the same
// ones (8 experts of 4096 x 14336, 24 tokens: 530 us per layer with all items starting at chunk 0, 446 us so; H = 2048: no
// difference).  What an XCD has at a time must differ in that chunk: an expert's tiles begin one XCD further on than those of
// the expert before.  An expert with more than 32 tokens has its token blocks of a row tile eight items apart, so that they
// read the same weights from one L2 at the same time (128 tokens on 8 experts of 4096 x 14336: 724 -> 700 us; 64 experts of
// 2048 x 1408, Zipf-skewed, 128 tokens: 195.5 -> 189.4 us, both with neighbouring blocks before).
//
// Any width that is a multiple of 8: rows and tokens beyond the end repeat the last one and are not stored; columns
// beyond the end of a row are zero in both operands.
#pragma once
#include "moe_internal.h"

namespace moe {

namespace wide {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kThreads = 1024, kWaves = 16;
constexpr int kToks = 32;                    // tokens of an item
constexpr int kStages = 3;                   // chunks in flight per workgroup
constexpr int kChunkBytes = 1024;            // 512 columns
constexpr int kRowLds = kChunkBytes + 16;    // (padding: sixteen rows' 16-byte words fall into sixteen bank groups)
constexpr int kTokLds = kToks * kRowLds;
constexpr int kItemLds = 64 * kRowLds + kWaves * 4 * 1024;   // tiles and partial results of an item of two row blocks; those of four share it
constexpr int kTokCap = kWideTokCap;

__device__ inline uint32_t f32_to_bf16_rne(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ inline f32x4 mfma(u32x4 a, u32x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The same value, but not one that the compiler may have worked with before: what an item's end derives from it is not kept
// in registers (or scratch memory) all through the loop.
__device__ __forceinline__ int here(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// TOK_LDS: the tokens of the list entries are in LDS (gate/up kernel, lists of up to kTokCap entries).  (A template
// argument: a global load that the walk might do would make every later wait in the loop one for all loads.)
// RB: blocks of 16 weight rows in an item (gate/up: the first half gate rows, the second half up rows).
template <bool GATEUP, bool TOK_LDS, int RB>
__device__ __forceinline__ void wide_body(const StreamArgs &a)
{
    constexpr int RPI = GATEUP ? 8 * RB : 16 * RB;   // output rows of an item
    constexpr int kTileLds = 16 * RB * kRowLds;
    static_assert(kChunkBytes == kWaves * 64, "a wavefront multiplies one block of 32 columns of a chunk");
    constexpr int kPart = kWaves * RB * 2 * 1024;          // partial results of an item
    constexpr bool OWN = kTileLds + kTokLds + kPart <= kItemLds;   // ... in LDS of their own, or in the place of the tiles
    static_assert(OWN || (kPart <= kItemLds && kTileLds + kTokLds <= kItemLds), "the item's LDS");
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char *const a_s = lds, *const b_s = lds + kTileLds;
    float *const part_s = (float *)(lds + (OWN ? kTileLds + kTokLds : 0));   // [token group][wavefront][row block][256] partial results
    const int A = a.T * a.k, n_cap = a.C + 1;
    int *const first_s = (int *)(lds + kItemLds);   // [active slot] its first item
    int *const m_s = first_s + n_cap, *const off_s = m_s + n_cap, *const slot_s = off_s + n_cap;
    uint16_t *const tok_s = (uint16_t *)(slot_s + n_cap);   // token of each list entry (A <= kTokCap)

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int G = gridDim.x, b = blockIdx.x;
    const int n_act = (int)*a.n_active;
    const int tiles = (a.R + RPI - 1) / RPI, tiles_sh = a.n_shared ? (a.R_sh + RPI - 1) / RPI : 0;
    const int nb_sh = (a.T + kToks - 1) / kToks, sh_items = a.n_shared * tiles_sh * nb_sh;   // (the shared experts' items come first)

    if (GATEUP && TOK_LDS)
        for (int i = tid; i < A; i += kThreads) tok_s[i] = (uint16_t)udiv_rcp(a.perm[i], a.k, a.rcp_k);
    for (int e = tid; e < n_act; e += kThreads) {
        const int c = a.active_slots[e];
        slot_s[e] = c;
        m_s[e] = a.slot_count[c];
        off_s[e] = a.slot_offset[c];
    }
    __syncthreads();
    if (w == 0) {
        // items before each active slot: row tiles x blocks of 32 tokens
        int base = sh_items;
        for (int e0 = 0; e0 < n_act; e0 += kWave) {
            const int e = e0 + lane;
            const int own = e < n_act ? (m_s[e] + kToks - 1) / kToks * tiles : 0;
            int inc = own;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int v = __shfl_up(inc, d, kWave);
                if (lane >= d) inc += v;
            }
            if (e < n_act) first_s[e] = base + inc - own;
            base += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
        if (lane == 0) first_s[n_act] = base;
    }
    __syncthreads();
    const int total = first_s[n_act];
    if (b >= total) return;

    // Item i: its expert, first row, first token, and the expert's tokens, first list entry (or act row) and place in
    // the pool.  Which workgroup (so: which XCD, i mod 8) gets a row tile: the token blocks of a tile lie eight items apart, on
    // one L2 at the same time; and an expert's tiles begin one XCD further on than those of the one before (see `prot`).
    struct Item { bool sh; int row0, tok0, m, off, slot; };
    auto decode = [&](int i) {
        Item it;
        int e, rem, nb, tl;
        it.sh = i < sh_items;
        if (it.sh) {
            e = i / (tiles_sh * nb_sh);
            rem = i - e * (tiles_sh * nb_sh);
            nb = nb_sh; tl = tiles_sh;
            it.m = a.T; it.off = e * a.T; it.slot = e;
        } else {
            e = -1;
            const int lane = here(threadIdx.x) & (kWave - 1);
            for (int e0 = 0; e0 < n_act; e0 += kWave) e += __popcll(__ballot(e0 + lane < n_act && first_s[e0 + lane] <= i));
            e = __builtin_amdgcn_readfirstlane(e);
            it.m = __builtin_amdgcn_readfirstlane(m_s[e]);
            it.off = __builtin_amdgcn_readfirstlane(off_s[e]);
            it.slot = __builtin_amdgcn_readfirstlane(slot_s[e]);
            rem = i - __builtin_amdgcn_readfirstlane(first_s[e]);
            nb = (it.m + kToks - 1) / kToks; tl = tiles;
        }
        int rt = rem, tb = 0;
        if (nb > 1) {
            const int q = rem / (8 * nb), r8 = rem - q * (8 * nb), gs = tl - 8 * q < 8 ? tl - 8 * q : 8;
            tb = r8 / gs;
            rt = 8 * q + r8 - tb * gs;
        }
        if (tl >= 8) {
            rt += e & 7;
            rt = rt < tl ? rt : rt - tl;
        }
        it.row0 = __builtin_amdgcn_readfirstlane(rt * RPI);
        it.tok0 = __builtin_amdgcn_readfirstlane(tb * kToks);
        return it;
    };

    // ---- the walk that loads: chunk pc of item pi is the next one to put in flight ----
    const unsigned char *pa[RB], *pb[2];   // this wavefront's weight rows (one of each block) and token rows
    int pi = b, pc = 0, pK2 = 0, pn = 0, prot = 0;   // (an item's chunks in turn from chunk prot on)
    auto prod_set = [&](int i) {
        const Item it = decode(i);
        const bool sh = it.sh;
        const int K = sh ? a.K_sh : a.K, R = sh ? a.R_sh : a.R;
        const int m = it.m, off = it.off;
        const size_t eoff = (size_t)it.slot * R * K;
        const uint16_t *const w0 = (sh ? a.s0 : a.w0) + eoff, *const w1 = (sh ? a.s1 : a.w1) + eoff;
        const uint16_t *const src = !GATEUP && sh ? a.bsrc_sh : a.bsrc;
        pK2 = 2 * K;
        pn = (pK2 + kChunkBytes - 1) / kChunkBytes;
        pc = 0;
        const int u = it.row0 >> (GATEUP ? 5 : 6);
        prot = K > kPanelMax ? (u + (u >> 3)) % pn : 0;
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            int r = it.row0 + 16 * (GATEUP ? j % (RB / 2) : j) + w;
            r = r < R ? r : R - 1;
            pa[j] = (const unsigned char *)((GATEUP && j >= RB / 2 ? w1 : w0) + (size_t)r * K);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            int t = it.tok0 + w + kWaves * j;
            t = t < m ? t : m - 1;
            int row = off + t;               // act row | list entry
            if (GATEUP) {
                if (sh) row = t;
                else row = TOK_LDS ? tok_s[row] : udiv_rcp(a.perm[row], a.k, a.rcp_k);
                row = __builtin_amdgcn_readfirstlane(row);
            }
            pb[j] = (const unsigned char *)(src + (size_t)row * K);
        }
    };
    u32x4 sa[kStages][RB], sb[kStages][2];
    int s_left[kStages];   // bytes of the row from the chunk's first column on
    auto issue = [&](int s) {
        const int pch = pc + prot < pn ? pc + prot : pc + prot - pn;
        const int o0 = pch * kChunkBytes, left = pK2 - o0, lane = here(threadIdx.x) & (kWave - 1);
        s_left[s] = left;
        const unsigned o = (unsigned)(o0 + (lane * 16 < left ? lane * 16 : left - 16));   // (lanes beyond the row's end re-read its last word)
#pragma unroll
        for (int j = 0; j < RB; ++j) sa[s][j] = __builtin_nontemporal_load((const u32x4 *)(pa[j] + o));
#pragma unroll
        for (int j = 0; j < 2; ++j) sb[s][j] = *(const u32x4 *)(pb[j] + o);
    };
    auto prod_advance = [&]() {
        if (pc + 1 < pn) {
            ++pc;
        } else if (pi + G < total) {
            pi += G;
            prod_set(pi);
        }   // (past the last item: its last chunk again, which nobody multiplies)
    };
    auto park = [&](int s) {
        const int lane = here(threadIdx.x) & (kWave - 1);
        if (s_left[s] < kChunkBytes) {
            const bool in = lane * 16 < s_left[s];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int j = 0; j < RB; ++j) sa[s][j][q] = in ? sa[s][j][q] : 0u;
#pragma unroll
                for (int j = 0; j < 2; ++j) sb[s][j][q] = in ? sb[s][j][q] : 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < RB; ++j) *(u32x4 *)(a_s + (w + kWaves * j) * kRowLds + lane * 16) = sa[s][j];
#pragma unroll
        for (int j = 0; j < 2; ++j) *(u32x4 *)(b_s + (w + kWaves * j) * kRowLds + lane * 16) = sb[s][j];
    };

    // ---- the walk that multiplies ----
    int ci = b, cc = 0;
    Item it = decode(ci);
    int cm = 0, cn = 0;
    auto cons_set = [&]() {
        cm = it.m;
        cn = (2 * (it.sh ? a.K_sh : a.K) + kChunkBytes - 1) / kChunkBytes;
        cc = 0;
    };
    // Wavefront w multiplies columns 32 w .. 32 w + 31 of every chunk, all row blocks and token groups of the item.
    f32x4 acc[RB][2];
    auto multiply = [&]() {
        const int ln = here(threadIdx.x) & (kWave - 1), at = (ln & 15) * kRowLds + w * 64 + (ln >> 4) * 16;
        const unsigned char *const ar = a_s + at, *const br = b_s + at;
        const bool two = cm - it.tok0 > 16;
        const u32x4 b0 = *(const u32x4 *)br;
        u32x4 b1 = {0u, 0u, 0u, 0u};
        if (two) b1 = *(const u32x4 *)(br + 16 * kRowLds);
#pragma unroll
        for (int j0 = 0; j0 < RB; j0 += 2) {
            u32x4 av[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) av[j] = *(const u32x4 *)(ar + (j0 + j) * (16 * kRowLds));
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[j0 + j][0] = mfma(av[j], b0, acc[j0 + j][0]);
                acc[j0 + j][1] = mfma(av[j], b1, acc[j0 + j][1]);
            }
            __builtin_amdgcn_sched_barrier(0);   // (no more reads ahead than the registers hold)
        }
    };
    // Element (row r, token t) of a 16 x 16 partial result lies in word (r / 4) * 64 + ((t + r / 4 + 4 * block) % 16) * 4 + r % 4:
    // what is read together, consecutive rows of one token, falls into banks of its own.
    auto post_partials = [&]() {
        const int gmax = cm - it.tok0 > 16 ? 2 : 1;
        const int ln = here(threadIdx.x) & (kWave - 1), n = ln & 15, g = ln >> 4;   // (the MFMA result's token; rows 4 g .. 4 g + 3)
#pragma unroll
        for (int gr = 0; gr < 2; ++gr)
            if (gr < gmax)
#pragma unroll
                for (int j = 0; j < RB; ++j)
                    *(f32x4 *)(part_s + ((gr * kWaves + w) * RB + j) * 256 + g * 64 + ((n + g + 4 * j) & 15) * 4) = acc[j][gr];
    };
    // ... and its sixteen partial results, added in wavefront order.
    auto total_of = [&](int block, int gr, int r, int t) {
        const float *p = part_s + (gr * kWaves * RB + block) * 256 + (r >> 2) * 64 + ((t + (r >> 2) + 4 * block) & 15) * 4 + (r & 3);
        float sum = 0.f;
#pragma unroll
        for (int i0 = 0; i0 < kWaves; i0 += 8) {
            float v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p[(i0 + i) * (RB * 256)];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum += v[i];
            __builtin_amdgcn_sched_barrier(0);
        }
        return sum;
    };
    auto finish = [&]() {
        const int tid = here(threadIdx.x);
        const bool sh = it.sh;
        const int R = sh ? a.R_sh : a.R;
        const size_t row0 = (size_t)it.off + it.tok0;
        if (GATEUP) {
            const int f = tid % RPI, t = tid / RPI;
            if (t < kToks && it.tok0 + t < cm && it.row0 + f < R) {
                const float gt = total_of(f >> 4, t >> 4, f & 15, t & 15), up = total_of(RB / 2 + (f >> 4), t >> 4, f & 15, t & 15);
                ((uint16_t *)(sh ? a.out_sh : a.out))[(row0 + t) * R + it.row0 + f] =
                    (uint16_t)f32_to_bf16_rne(gt / (1.f + expf(-gt)) * up);
            }
        } else {
            const int r = tid % RPI;
#pragma unroll
            for (int t = tid / RPI; t < kToks; t += kThreads / RPI)
                if (it.tok0 + t < cm && it.row0 + r < R)
                    ((float *)(sh ? a.out_sh : a.out))[(row0 + t) * R + it.row0 + r] = total_of(r >> 4, t >> 4, r & 15, t & 15);
        }
    };

    cons_set();
    prod_set(pi);
#pragma unroll
    for (int s = 0; s < kStages; ++s) {
        issue(s);
        prod_advance();
    }
    auto step = [&](int s) {
        park(s);
        issue(s);
        prod_advance();
        __syncthreads();
        if (cc == 0)
#pragma unroll
            for (int j = 0; j < RB; ++j) acc[j][0] = acc[j][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
        multiply();
        const bool last = ++cc == cn;
        if (OWN && last) post_partials();
        __syncthreads();
        if (last) {
            if (!OWN) {
                post_partials();
                __syncthreads();
            }
            finish();
            if (!OWN) __syncthreads();   // (OWN: the next ones are written behind the next step's first barrier)
            if (ci + G < total) {
                ci += G;
                it = decode(ci);
                cons_set();
            }
        }
    };
    // chunks of this workgroup's items (shared experts' items come first).  The first step is peeled off and the
    // loop goes in threes, so that the compiler's count of the loads in flight is exact: a park waits for its own chunk.
    const int n_sh = sh_items > b ? (sh_items - b + G - 1) / G : 0, n_all = (total - b + G - 1) / G;
    const int chunks = n_sh * ((2 * a.K_sh + kChunkBytes - 1) / kChunkBytes) + (n_all - n_sh) * ((2 * a.K + kChunkBytes - 1) / kChunkBytes);
    step(0);
    int c = 1;
    static_assert(kStages == 3, "the loop below");
    for (; c + 2 < chunks; c += 3) {
        step(1);
        step(2);
        step(0);
    }
    if (c < chunks) step(1);
    if (c + 1 < chunks) step(2);
}

}  // namespace wide

}  // namespace moe
