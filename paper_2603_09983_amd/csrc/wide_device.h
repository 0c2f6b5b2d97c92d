// Expert FFN of larger batches (use_wide_kernels(); Sec. 2.2 last line, experts as in App. D):
//      act = silu(W_gate x) * (W_up x)        (gate/up kernel)
//      o   = W_down act                       (down kernel)
//
// The small-batch kernels (stream.hip) keep an expert's B operand, all columns of up to 32 tokens, in the registers
// of sixteen wavefronts and stream whole weight rows past it.  With more tokens per expert, or with two token groups and
// rows of several panels, that operand has to come again for every tile.  Here an item is 64 weight rows (32 gate rows
// on 32 up rows, or 64 down rows) against 32 tokens of one expert's list; both operands pass through LDS in chunks of
// 512 columns, every load instruction one row's consecutive kilobyte, and the accumulators stay in registers for the
// whole contraction.  Bound: HBM for the weights.  An expert's weights are read once for each 32 of its tokens, and the
// L2s do not keep them in between (FETCH_SIZE, 8 experts of 4096 x 14336: gate/up 1.92 GB for 1.88 GB of weights at 64 tokens,
// all lists within 32; 2.77 GB at 128 tokens, 12 blocks on 8 experts, where 2.82 GB would be no reuse at all).
//
// One workgroup of sixteen wavefronts per CU takes items b, b + G, .. and keeps three chunks in flight, across items
// (3 x 64 KB of weights).
//
// The order of the sums is fixed: four parts of the columns (128 of every chunk's 512 each, chunk after chunk), added through
// LDS.  It follows from the row and the widths alone: a token's outputs have the same bits whatever else is in the batch,
// wherever the item lies in the list and with 64 or 32 rows to an item.
//
// Rows of several panels (K > kPanelMax) start at a chunk that follows from the row: with rows of 8 KB and more all rows'
// kilobytes of one chunk lie in few of an L2's sixteen channels, and workgroups that start together would all be in the same
// ones (8 experts of 4096 x 14336, 24 tokens: 530 us per layer with all items starting at chunk 0, 441 us so; H = 2048: no
// difference).  What an XCD has at a time must differ in that chunk: an expert's tiles begin one XCD further on than those of
// the expert before.  An expert with more than 32 tokens has its token blocks of a row tile eight items apart, on one XCD, with
// the same first chunk (128 tokens on 8 experts of 4096 x 14336: 725 us with neighbouring blocks at chunks of their own, 715 so).
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
constexpr int kRing = 8, kRingLds = kRing * 32;   // items between the walk that loads and the one that multiplies
constexpr int kItemLds = 96 * kRowLds + kWaves * 2 * 1024 + kRingLds;   // tiles and partial results of an item of four row blocks; the ring
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
    constexpr int GW = RB / 2;                       // token groups that a wavefront multiplies (with two row blocks each group has its own)
    static_assert((RB == 2 || RB == 4) && kTileLds + kTokLds + kWaves * GW * 1024 + kRingLds <= kItemLds, "wavefronts; the item's LDS");
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char *const a_s = lds, *const b_s = lds + kTileLds;
    float *const part_s = (float *)(lds + kTileLds + kTokLds);   // [wavefront][its token group][256] partial results
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
    const unsigned rcp_sh = sh_items ? rcp32((unsigned)(tiles_sh * nb_sh)) : 0u;

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
    // one XCD; and an expert's tiles begin one XCD further on than those of the one before (see `prot`).
    struct Item { bool sh; int row0, tok0, m, off, slot; };
    auto decode = [&](int i) {
        Item it;
        int e, rem, nb, tl;
        it.sh = i < sh_items;
        if (it.sh) {
            e = udiv_rcp(i, tiles_sh * nb_sh, rcp_sh);
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
            // eight row tiles by nb blocks at a time; the tiles that are left (fewer than eight) have their blocks as neighbours
            const int whole = (tl & ~7) * nb, y = rem < whole ? rem >> 3 : rem - whole, d = y / nb;
            tb = y - d * nb;
            rt = rem < whole ? 8 * d + (rem & 7) : (tl & ~7) + d;
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
    // (The walk that multiplies follows three chunks behind and takes the items from a ring in LDS: at most four are under
    // way, and a place is written again several barriers after it was read.)
    int *const ring_s = (int *)(lds + kItemLds - kRingLds);
    int pord = 0;
    auto prod_put = [&](const Item &it) {
        if (tid == 0) {
            int *const r = ring_s + (pord & (kRing - 1)) * 8;
            r[0] = it.sh; r[1] = it.row0; r[2] = it.tok0; r[3] = it.m; r[4] = it.off;
        }
        ++pord;
    };
    int pi = b, pc = 0, pK2 = 0, pn = 0, prot = 0;   // (an item's chunks in turn from chunk prot on)
    auto prod_set = [&](const Item &it) {
        prod_put(it);
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
            prod_set(decode(pi));
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
    int ci = b, cc = 0, cord = 0;
    Item it = decode(ci);
    int cm = 0, cn = 0;
    auto cons_set = [&]() {
        cm = it.m;
        cn = (2 * (it.sh ? a.K_sh : a.K) + kChunkBytes - 1) / kChunkBytes;
        cc = 0;
    };
    // Wavefront w multiplies row block w % RB by GW token groups, the column part kq = w / 4 (128 columns) of every chunk.
    const int rb = w % RB, g0 = RB == 2 ? w / 2 % 2 : 0, kq = w / 4;
    f32x4 acc[GW];
    auto multiply = [&]() {
        const int ln = here(threadIdx.x) & (kWave - 1), at = (ln & 15) * kRowLds + kq * (kChunkBytes / 4) + (ln >> 4) * 16;
        const unsigned char *const ar = a_s + 16 * rb * kRowLds + at, *const br = b_s + 16 * g0 * kRowLds + at;
        if (g0 == 1 && cm - it.tok0 <= 16) return;
        u32x4 av[4], bv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            av[j] = *(const u32x4 *)(ar + j * 64);
            bv[j] = *(const u32x4 *)(br + j * 64);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[0] = mfma(av[j], bv[j], acc[0]);
        if (GW == 2 && cm - it.tok0 > 16) {
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[j] = *(const u32x4 *)(br + 16 * kRowLds + j * 64);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[GW - 1] = mfma(av[j], bv[j], acc[GW - 1]);
        }
    };
    // Element (row r, token t) of a 16 x 16 partial result lies in word (r / 4) * 64 + ((t + r / 4 + 4 * block) % 16) * 4 + r % 4:
    // what is read together, consecutive rows of one token, falls into banks of its own.
    auto post_partials = [&]() {
        const int ln = here(threadIdx.x) & (kWave - 1), n = ln & 15, g = ln >> 4;   // (the MFMA result's token; rows 4 g .. 4 g + 3)
#pragma unroll
        for (int i = 0; i < GW; ++i) *(f32x4 *)(part_s + (w * GW + i) * 256 + g * 64 + ((n + g + 4 * rb) & 15) * 4) = acc[i];
    };
    // ... and its four partial results, added in the order of the column parts.
    auto total_of = [&](int block, int gr, int r, int t) {
        const float *p = part_s + (RB == 2 ? gr * 2 + block : block * 2 + gr) * 256 + (r >> 2) * 64 + ((t + (r >> 2) + 4 * block) & 15) * 4 + (r & 3);
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = p[i * (4 * GW * 256)];
        return v[0] + v[1] + v[2] + v[3];
    };
    // (every wavefront's partial results are there; the next ones are written behind another barrier)
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
    prod_set(it);
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
            for (int i = 0; i < GW; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        multiply();
        const bool last = ++cc == cn;
        if (last) post_partials();
        __syncthreads();
        if (last) {
            finish();
            if (ci + G < total) {
                ci += G;
                const int *const r = ring_s + (++cord & (kRing - 1)) * 8;
                it.sh = __builtin_amdgcn_readfirstlane(r[0]) != 0;
                it.row0 = __builtin_amdgcn_readfirstlane(r[1]);
                it.tok0 = __builtin_amdgcn_readfirstlane(r[2]);
                it.m = __builtin_amdgcn_readfirstlane(r[3]);
                it.off = __builtin_amdgcn_readfirstlane(r[4]);
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
