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
// (3 x 64 KB of weights; two workgroups of eight wavefronts with two chunks of 32 KB each measured the same).  Wavefront w multiplies row block w % 4 with the column part w / 4 of the chunk; the four partial results
// are added through LDS, in a fixed order, while the next chunk is parked.
//
// An item starts at a chunk of its own, (item / 8) mod chunks: with rows of 4 or 8 KB all rows' kilobytes of one chunk
// lie in a quarter or an eighth of an L2's sixteen channels, and workgroups that start together would all be in the same
// ones (items 8 apart run on the same L2).  Loads alone, 554 MB of gate/up weights with H = 2048: 100 us with all items
// starting at chunk 0, 90 us so; 1.88 GB with H = 4096: 350 and 298 us.
//
// Measured (kernels, gate/up + down): 64 tokens, 8 experts of 4096 x 14336: 321 + 163 us (5.9 and 5.7 TB/s), 1048 us in
// the general kernel; 256 tokens, 48 experts of 2048 x 1408, a mean of 24 tokens each: 112 + 73 us, 247 + 128 us in the
// streaming kernels, which reload the B operand and drain their loads for every pass over a tile.  At 128 tokens (a mean
// of 12) those take 88 + 49 us against 99 + 58 here: the rules that choose are use_wide_kernels() and either_kernel.
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

// TOK_LDS: the tokens of the list entries are in LDS (gate/up kernel, lists of up to kTokCap entries).  (A template
// argument: a global load that the walk might do would make every later wait in the loop one for all loads.)
// RB: blocks of 16 weight rows in an item (gate/up: the first half gate rows, the second half up rows).
template <bool GATEUP, bool TOK_LDS, int RB>
__device__ __forceinline__ void wide_body(const StreamArgs &a)
{
    constexpr int RPI = GATEUP ? 8 * RB : 16 * RB;   // output rows of an item
    constexpr int KQ = kWaves / RB;                  // parts that the columns of a chunk are split into
    constexpr int KB = kChunkBytes / 64 / KQ;        // 32-wide column blocks of a part
    constexpr int kTileLds = 16 * RB * kRowLds;
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char *const a_s = lds, *const b_s = lds + kTileLds;
    float *const red_s = (float *)(lds + kTileLds + kTokLds);   // [wavefront][token group][256] partial results
    const int A = a.T * a.k, n_cap = a.n_shared + a.C + 1;
    int *const first_s = (int *)(red_s + kWaves * 2 * 256);   // [entry] its first item (entries: shared experts, active slots)
    int *const m_s = first_s + n_cap, *const off_s = m_s + n_cap, *const slot_s = off_s + n_cap;
    uint16_t *const tok_s = (uint16_t *)(slot_s + n_cap);   // token of each list entry (A <= kTokCap)

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int n = lane & 15, g = lane >> 4;
    const int G = gridDim.x, b = blockIdx.x;
    const int n_act = (int)*a.n_active, n_ent = a.n_shared + n_act;
    const int tiles = (a.R + RPI - 1) / RPI, tiles_sh = a.n_shared ? (a.R_sh + RPI - 1) / RPI : 0;

    if (GATEUP && TOK_LDS)
        for (int i = tid; i < A; i += kThreads) tok_s[i] = (uint16_t)udiv_rcp(a.perm[i], a.k, a.rcp_k);
    for (int e = tid; e < n_ent; e += kThreads) {
        const int c = e < a.n_shared ? e : a.active_slots[e - a.n_shared];
        slot_s[e] = c;
        m_s[e] = e < a.n_shared ? a.T : a.slot_count[c];
        off_s[e] = e < a.n_shared ? e * a.T : a.slot_offset[c];
    }
    __syncthreads();
    if (w == 0) {
        // items before each entry: row tiles x blocks of 32 tokens
        int base = 0;
        for (int e0 = 0; e0 < n_ent; e0 += kWave) {
            const int e = e0 + lane;
            const int own = e < n_ent ? (m_s[e] + kToks - 1) / kToks * (e < a.n_shared ? tiles_sh : tiles) : 0;
            int inc = own;
#pragma unroll
            for (int d = 1; d < kWave; d <<= 1) {
                const int v = __shfl_up(inc, d, kWave);
                if (lane >= d) inc += v;
            }
            if (e < n_ent) first_s[e] = base + inc - own;
            base += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
        if (lane == 0) first_s[n_ent] = base;
    }
    __syncthreads();
    const int total = first_s[n_ent];
    if (b >= total) return;

    // Item i: its entry (expert), row tile and token block.  The blocks of a row tile are neighbours.
    struct Item { int e, row0, tok0; };
    auto decode = [&](int i) {
        int e = -1;
        for (int e0 = 0; e0 < n_ent; e0 += kWave) e += __popcll(__ballot(e0 + lane < n_ent && first_s[e0 + lane] <= i));
        e = __builtin_amdgcn_readfirstlane(e);
        const int nb = (__builtin_amdgcn_readfirstlane(m_s[e]) + kToks - 1) / kToks;
        const int rem = i - __builtin_amdgcn_readfirstlane(first_s[e]);
        const int rt = nb == 1 ? rem : rem / nb;
        return Item{e, rt * RPI, (rem - rt * nb) * kToks};
    };

    // ---- the walk that loads: chunk pc of item pi is the next one to put in flight ----
    const unsigned char *pa[RB], *pb[2];   // this wavefront's weight rows (one of each block) and token rows
    int pi = b, pc = 0, pK2 = 0, pn = 0, prot = 0;   // (an item's chunks in turn from chunk prot on)
    auto prod_set = [&](int i) {
        const Item it = decode(i);
        const bool sh = it.e < a.n_shared;
        const int K = sh ? a.K_sh : a.K, R = sh ? a.R_sh : a.R;
        const int m = __builtin_amdgcn_readfirstlane(m_s[it.e]), off = __builtin_amdgcn_readfirstlane(off_s[it.e]);
        const size_t eoff = (size_t)__builtin_amdgcn_readfirstlane(slot_s[it.e]) * R * K;
        const uint16_t *const w0 = (sh ? a.s0 : a.w0) + eoff, *const w1 = (sh ? a.s1 : a.w1) + eoff;
        const uint16_t *const src = !GATEUP && sh ? a.bsrc_sh : a.bsrc;
        pK2 = 2 * K;
        pn = (pK2 + kChunkBytes - 1) / kChunkBytes;
        pc = 0;
        prot = (i >> 3) % pn;
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
        const int o0 = pch * kChunkBytes, left = pK2 - o0;
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
    const int rb = w % RB, kq = w / RB;
    int ci = b, cc = 0;
    Item it = decode(ci);
    int cm = 0, cn = 0;
    auto cons_set = [&]() {
        cm = __builtin_amdgcn_readfirstlane(m_s[it.e]);
        cn = (2 * (it.e < a.n_shared ? a.K_sh : a.K) + kChunkBytes - 1) / kChunkBytes;
        cc = 0;
    };
    f32x4 acc[2];
    auto multiply = [&]() {
        const unsigned char *const ar = a_s + (16 * rb + n) * kRowLds + kq * (64 * KB) + g * 16;
        const unsigned char *const br = b_s + n * kRowLds + kq * (64 * KB) + g * 16;
        u32x4 av[KB], bv[KB];
#pragma unroll
        for (int j = 0; j < KB; ++j) {
            av[j] = *(const u32x4 *)(ar + j * 64);
            bv[j] = *(const u32x4 *)(br + j * 64);
        }
#pragma unroll
        for (int j = 0; j < KB; ++j) acc[0] = mfma(av[j], bv[j], acc[0]);
        if (cm - it.tok0 > 16) {
#pragma unroll
            for (int j = 0; j < KB; ++j) bv[j] = *(const u32x4 *)(br + 16 * kRowLds + j * 64);
#pragma unroll
            for (int j = 0; j < KB; ++j) acc[1] = mfma(av[j], bv[j], acc[1]);
        }
    };
    // The partial results of each element (wavefronts rb, rb + RB, ..), added in that order.
    // Element (row r, token t) of a 16 x 16 result sits at ((r / 4) * 16 + t) * 4 + r % 4.
    auto total_of = [&](int block, int gr, int r, int t) {
        const float *p = red_s + (block * 2 + gr) * 256 + ((r >> 2) * 16 + t) * 4 + (r & 3);
        float v[KQ];
#pragma unroll
        for (int i = 0; i < KQ; ++i) v[i] = p[i * (RB * 512)];
#pragma unroll
        for (int i = 1; i < KQ; ++i) v[0] += v[i];
        return v[0];
    };
    // (every wavefront's partial results are there; the next ones are written behind another barrier)
    auto finish = [&]() {
        const bool sh = it.e < a.n_shared;
        const int R = sh ? a.R_sh : a.R;
        const size_t row0 = (size_t)__builtin_amdgcn_readfirstlane(off_s[it.e]) + it.tok0;
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
        if (cc == 0) acc[0] = acc[1] = (f32x4){0.f, 0.f, 0.f, 0.f};
        multiply();
        const bool last = ++cc == cn;
        if (last)
#pragma unroll
            for (int gr = 0; gr < 2; ++gr) *(f32x4 *)(red_s + (w * 2 + gr) * 256 + lane * 4) = acc[gr];
        __syncthreads();
        if (last) {
            finish();
            if (ci + G < total) {
                ci += G;
                it = decode(ci);
                cons_set();
            }
        }
    };
    // chunks of this workgroup's items (shared experts' items come first).  The first step is peeled off and the
    // loop goes in threes, so that the compiler's count of the loads in flight is exact: a park waits for its own chunk.
    const int n_sh = first_s[a.n_shared] > b ? (first_s[a.n_shared] - b + G - 1) / G : 0, n_all = (total - b + G - 1) / G;
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
