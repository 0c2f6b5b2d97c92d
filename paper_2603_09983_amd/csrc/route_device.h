// Device-side pieces of the routing steps (Top-k and gate of one token or of four per wavefront, histogram, slot
// lookup, miss list and per-slot lists of a whole batch per workgroup), shared by the routing kernel and
// by the gate/up kernel that does the routing itself.  Included inside an unnamed namespace of each
// translation unit.
#pragma once
#include "moe_internal.h"

namespace moe {

namespace {

constexpr int kRouteThreads = 1024;
constexpr int kRouteWaves = kRouteThreads / kWave;
constexpr int kLdsCopy = 4096;  // assignments whose ids are mirrored in LDS

__device__ inline float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ inline float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

// LDS and global pointers carry their address space: a generic pointer would turn every access into
// a flat instruction, and the dependent LDS reads below would each cost a trip through the memory
// pipeline instead of an LDS access.
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) int lds_i32;
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const f32x4v lds_f32x4;
typedef __attribute__((address_space(1))) int32_t g_i32;
typedef __attribute__((address_space(1))) float g_f32;
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const f32x4v g_f32x4;
typedef __attribute__((address_space(1))) const u32x2v g_u32x2;

// Value of v in the lane n places further on inside the row of 16 lanes, wrapping round (register to
// register, no trip through LDS): data-parallel-primitive control row_ror:n = 0x120 + n.
template <int N>
__device__ __forceinline__ unsigned row_rotate(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + N, 0xf, 0xf, false);
}

// Maximum of x over the 64 lanes of a wavefront (all of them active), in every lane: four rotations inside the rows of
// sixteen, then the rows exchanged pairwise and by halves.  All in vector registers: through four readlanes and scalar maxima the
// value changes register file twice, and each of the k steps of a ranking took 0.16 us instead of 0.07.
__device__ __forceinline__ unsigned wave_max_u32(unsigned x)
{
    unsigned y;
    y = row_rotate<1>(x); x = x > y ? x : y;
    y = row_rotate<2>(x); x = x > y ? x : y;
    y = row_rotate<4>(x); x = x > y ? x : y;
    y = row_rotate<8>(x); x = x > y ? x : y;
    const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = r[0] > r[1] ? r[0] : r[1];
    const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return h[0] > h[1] ? h[0] : h[1];
}

// Sum of x over the 64 lanes, likewise.
__device__ __forceinline__ unsigned wave_sum_u32(unsigned x)
{
    x += row_rotate<1>(x);
    x += row_rotate<2>(x);
    x += row_rotate<4>(x);
    x += row_rotate<8>(x);
    return (unsigned)__builtin_amdgcn_readlane((int)x, 0) + (unsigned)__builtin_amdgcn_readlane((int)x, 16) +
           (unsigned)__builtin_amdgcn_readlane((int)x, 32) + (unsigned)__builtin_amdgcn_readlane((int)x, 48);
}

// One wavefront picks the Top-k of the E logits of one token, best first: k times the maximum over the
// wavefront, ties to the lower expert id, the winner taken out.  Logits are compared as unsigned keys
// that order like the floats (-0 counted as +0; key 0 = taken or no expert, below every float).  The
// gate is exp(s - s_max) normalised over the k, summed in rank order.  Lane l owns experts l, l+64, ...;
// the caller has put the logits into `lg` (LDS private to the wavefront: E floats, NaN replaced by -inf; overwritten).
// Needs k <= E and all 64 lanes active.  Returns the gate weight of the pick of rank `lane` (lanes >= k: unspecified); with
// idx_out null the ids are wanted in LDS only, and there is no gate.
//
// Bound by the latency of the k dependent steps (about a hundred cycles each), so a step does nothing but find the winner and
// take it out: the winner's own lane notes the rank, and the picks are put in order through LDS at the end.  Six of 64
// experts with the gate: 0.95 -> 0.55 us.
template <int NLOC>
__device__ __forceinline__ float wave_topk_gate_n(int E, int k, int32_t *idx_out_, lds_i32 *idx_lds,
                                                  float *w_out_, lds_f32 *lg)
{
    g_i32 *idx_out = (g_i32 *)(uintptr_t)idx_out_;
    g_f32 *w_out = (g_f32 *)(uintptr_t)w_out_;
    const int lane = threadIdx.x & (kWave - 1);
    unsigned key[NLOC];
    float val[NLOC];
    int rank[NLOC];
#pragma unroll
    for (int i = 0; i < NLOC; ++i) {
        const int e = lane + kWave * i;
        float f = e < E ? lg[e] : 0.f;
        f = f == 0.f ? 0.f : f;
        const unsigned u = __float_as_uint(f);
        val[i] = f;
        key[i] = e < E ? ((u & 0x80000000u) ? ~u : (u | 0x80000000u)) : 0u;
        rank[i] = k;
    }
    for (int j = 0; j < k; ++j) {
        unsigned m = key[0];
#pragma unroll
        for (int i = 1; i < NLOC; ++i) m = m > key[i] ? m : key[i];
        const unsigned best = wave_max_u32(m);
        // lowest id among the experts that hold it: the lowest i that has one, then the lowest lane
        bool open = true;
#pragma unroll
        for (int i = 0; i < NLOC; ++i) {
            const unsigned long long bal = __ballot(key[i] == best);
            const int win = open && bal ? __ffsll((long long)bal) - 1 : -1;
            open = open && bal == 0ull;
            if (lane == win) {
                rank[i] = j;
                key[i] = 0u;
            }
        }
    }
    // (LDS operations of one wavefront execute in order: every logit has been read above)
#pragma unroll
    for (int i = 0; i < NLOC; ++i) {
        if (rank[i] < k) {
            const int e = lane + kWave * i;
            lg[rank[i]] = val[i];
            if (idx_lds) idx_lds[rank[i]] = e;
            if (idx_out_) idx_out[rank[i]] = e;
        }
    }
    __builtin_amdgcn_wave_barrier();
    if (!idx_out_) return 0.f;
    const float my_s = lane < k ? lg[lane] : 0.f;
    const float smax = __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(my_s), 0));
    const float ex = lane < k ? __expf(my_s - smax) : 0.f;
    float den = 0.f;
    for (int j = 0; j < k; ++j) den += __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(ex), j));
    const float gate = ex / den;
    if (lane < k) w_out[lane] = gate;
    return gate;
}

__device__ __forceinline__ void wave_topk_gate(int E, int k, int32_t *idx_out, lds_i32 *idx_lds, float *w_out,
                                               lds_f32 *lg)
{
    if (E <= kWave) wave_topk_gate_n<1>(E, k, idx_out, idx_lds, w_out, lg);
    else if (E <= 2 * kWave) wave_topk_gate_n<2>(E, k, idx_out, idx_lds, w_out, lg);
    else if (E <= 4 * kWave) wave_topk_gate_n<4>(E, k, idx_out, idx_lds, w_out, lg);
    else wave_topk_gate_n<kMaxEPL>(E, k, idx_out, idx_lds, w_out, lg);
}

// Four tokens to a wavefront, a row of sixteen lanes each (E <= 64, k <= 16; tokens t0 .. t0 + 3, those below t_end): waits, at
// most `spin` polls, until their logits in `src` carry `tag`, and ranks them like wave_topk_gate_n, same order, same gate.  Lane l of a
// row owns experts l, l + 16, l + 32, l + 48.  Returns false if the wait ran out.
// For batches of which every wavefront would have tokens: sixteen wavefronts that rank one token each share four vector units, and
// a step costs half as many instructions a token so (17 tokens on 64 experts of 2048 x 1408, two a wavefront before: the layer 118.9 ->
// 117.3 us; 1 to 16 tokens, one a wavefront, gain nothing: 25.6 | 25.8 us at one, 74.5 | 75.0 at nine).  E <= 64 because a lane holds
// four experts; more would take eight keys a lane, which was not measured: there one token to a wavefront stays.
__device__ __forceinline__ bool rows_topk_gate(int E, int k, int t0, int t_end, const unsigned long long *src_, unsigned tag, int spin,
                                               lds_i32 *idx_lds, int32_t *idx_out_, float *w_out_)
{
    typedef __attribute__((address_space(1))) const unsigned long long g_u64;
    const int lane = threadIdx.x & (kWave - 1), l = lane & 15, t = t0 + (lane >> 4);
    const bool on = t < t_end;
    g_u64 *const src = (g_u64 *)(uintptr_t)src_ + (size_t)(on ? t : t0) * E;
    unsigned long long v[4];
    bool in_time = true;
    for (int polls = 0;;) {
        bool late = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = l + 16 * i;
            v[i] = __hip_atomic_load(src + (e < E ? e : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) late = late || (unsigned)(v[i] >> 32) != tag;
        if (__ballot(late) == 0ull) break;
        if (++polls > spin) {
            in_time = false;
            break;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    unsigned key[4], my_key = 0x80000000u;
    int my_e = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float f = __uint_as_float((unsigned)v[i]);
        f = f == f ? f : -INFINITY;   // NaN cannot win a comparison; rank it last
        f = f == 0.f ? 0.f : f;
        const unsigned u = __float_as_uint(f);
        key[i] = l + 16 * i < E ? ((u & 0x80000000u) ? ~u : (u | 0x80000000u)) : 0u;
    }
    auto row_max = [](unsigned x) __attribute__((always_inline)) {
        unsigned y;
        y = row_rotate<1>(x); x = x > y ? x : y;
        y = row_rotate<2>(x); x = x > y ? x : y;
        y = row_rotate<4>(x); x = x > y ? x : y;
        y = row_rotate<8>(x); return x > y ? x : y;
    };
    for (int j = 0; j < k; ++j) {
        const unsigned a = key[0] > key[1] ? key[0] : key[1], b = key[2] > key[3] ? key[2] : key[3];
        const unsigned best = row_max(a > b ? a : b);
        unsigned mine = 0u;   // 64 - the lowest id of this lane's that holds the maximum
#pragma unroll
        for (int i = 3; i >= 0; --i) mine = key[i] == best ? 64u - (unsigned)(l + 16 * i) : mine;
        const int e = 64 - (int)row_max(mine);
#pragma unroll
        for (int i = 0; i < 4; ++i) key[i] = l + 16 * i == e ? 0u : key[i];
        my_key = l == j ? best : my_key;
        my_e = l == j ? e : my_e;
    }
    if (on && l < k) idx_lds[t * k + l] = my_e;
    if (!idx_out_) return in_time;
    const float my_s = __uint_as_float((my_key & 0x80000000u) ? (my_key ^ 0x80000000u) : ~my_key);
    const float ex = l < k ? __expf(my_s - __shfl(my_s, lane & 48, kWave)) : 0.f;
    float den = 0.f;
    for (int j = 0; j < k; ++j) den += __shfl(ex, (lane & 48) + j, kWave);
    if (on && l < k) {
        ((g_i32 *)(uintptr_t)idx_out_)[(size_t)t * k + l] = my_e;
        ((g_f32 *)(uintptr_t)w_out_)[(size_t)t * k + l] = ex / den;
    }
    return in_time;
}

// The bias of expert e, the same in all lanes, by a vector load: a scalar one would be waited for, cold, before the row
// addresses behind it in the scalar unit's queue (5 tokens with a bias, one shared expert of 5632: 1.9 % of the layer's 50 us).
__device__ __forceinline__ float load_bias(const float *bias, int e)
{
    asm volatile("" : "+v"(e));
    return *(g_f32 *)(uintptr_t)(bias + e);
}

// One lane's part of the dot product of a router row with a token's hidden row: columns 4 lane, 4 lane + 256, .. in
// ascending order.  The loads of up to 2048 columns are on their way together; where fewer are left, a lane beyond the
// row's end re-reads its last columns and adds nothing.  (A plain loop fetches the columns of an H below 2048 one kilobyte
// after the other: H = 2040, 7 tokens, 2.7 us instead of 1.2.)
__device__ __forceinline__ float wave_dot(const float *wrow, const uint16_t *xr, int H)
{
    const int lane = threadIdx.x & (kWave - 1);
    float acc = 0.f;
    auto term = [](f32x4v wv, u32x2v xv) __attribute__((always_inline)) {
        return wv.x * bf16_lo(xv.x) + wv.y * bf16_hi(xv.x) + wv.z * bf16_lo(xv.y) + wv.w * bf16_hi(xv.y);
    };
    int h0 = 0;
    for (; h0 + 8 * kWave * 4 <= H; h0 += 8 * kWave * 4) {
        f32x4v wv[8];
        u32x2v xv[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            wv[i] = *(g_f32x4 *)(uintptr_t)(wrow + h0 + lane * 4 + i * kWave * 4);
            xv[i] = *(g_u32x2 *)(uintptr_t)(xr + h0 + lane * 4 + i * kWave * 4);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) acc += term(wv[i], xv[i]);
    }
    if (h0 < H) {
        f32x4v wv[8] = {};
        u32x2v xv[8] = {};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (h0 + i * kWave * 4 >= H) break;
            const int h = h0 + i * kWave * 4 + lane * 4;
            const unsigned o = (unsigned)(h < H ? h : H - 4);
            wv[i] = *(g_f32x4 *)((uintptr_t)wrow + o * 4u);
            xv[i] = *(g_u32x2 *)((uintptr_t)xr + o * 2u);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (h0 + i * kWave * 4 >= H) break;
            const float p = term(wv[i], xv[i]);
            acc += h0 + i * kWave * 4 + lane * 4 < H ? p : 0.f;
        }
    }
    return acc;
}

// The same for four tokens at once (rows xr[0..3]): each gets the sum that wave_dot gives it.  The router row is fetched once
// for the four, 1024 columns at a time.
__device__ __forceinline__ void wave_dot4(const float *wrow, const uint16_t *const (&xr)[4], int H, float (&acc)[4])
{
    const int lane = threadIdx.x & (kWave - 1);
    constexpr int kStep = 4 * kWave * 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = 0.f;
    auto add = [&](const f32x4v &wv, const u32x2v &xv, float &a, bool in) __attribute__((always_inline)) {
        const float p = wv.x * bf16_lo(xv.x) + wv.y * bf16_hi(xv.x) + wv.z * bf16_lo(xv.y) + wv.w * bf16_hi(xv.y);
        a += in ? p : 0.f;
    };
    int h0 = 0;
#pragma unroll 2
    for (; h0 + kStep <= H; h0 += kStep) {
        f32x4v wv[4];
        u32x2v xv[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            wv[i] = *(g_f32x4 *)(uintptr_t)(wrow + h0 + lane * 4 + i * kWave * 4);
#pragma unroll
            for (int t = 0; t < 4; ++t) xv[i][t] = *(g_u32x2 *)(uintptr_t)(xr[t] + h0 + lane * 4 + i * kWave * 4);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < 4; ++t) add(wv[i], xv[i][t], acc[t], true);
    }
    if (h0 < H) {
        f32x4v wv[4] = {};
        u32x2v xv[4][4] = {};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (h0 + i * kWave * 4 >= H) break;
            const int h = h0 + i * kWave * 4 + lane * 4;
            const unsigned o = (unsigned)(h < H ? h : H - 4);
            wv[i] = *(g_f32x4 *)((uintptr_t)wrow + o * 4u);
#pragma unroll
            for (int t = 0; t < 4; ++t) xv[i][t] = *(g_u32x2 *)((uintptr_t)xr[t] + o * 2u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (h0 + i * kWave * 4 >= H) break;
#pragma unroll
            for (int t = 0; t < 4; ++t) add(wv[i], xv[i][t], acc[t], h0 + i * kWave * 4 + lane * 4 < H);
        }
    }
}

// logits of one token in LDS: E floats, each wavefront's row starting on a multiple of four
__host__ __device__ inline int lg_stride(int E) { return (E + 3) & ~3; }


// hist[e] = number of assignments naming expert e (LDS integer atomics).
__device__ void block_histogram(const int32_t *idx, int A, int E, int32_t *hist, lds_i32 *hist_s)
{
    for (int e = threadIdx.x; e < E; e += blockDim.x) hist_s[e] = 0;
    __syncthreads();
    for (int a = threadIdx.x; a < A; a += blockDim.x) {
        int e = idx[a];
        if ((unsigned)e < (unsigned)E) __hip_atomic_fetch_add(&hist_s[e], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += blockDim.x) hist[e] = hist_s[e];
}

// Histogram (optional), slot lookup, ascending miss list, per-slot assignment lists and the
// list of active slots, by one workgroup.  idx / slot_table may point to LDS copies.
//   hist == nullptr: no histogram.   slot_table == nullptr: slot_idx is an input (lists only).
//   block: 16 or 32, the tokens of a block as n_blocks counts them.
// LDS: hist_s[E], cnt_s[kRouteWaves][C], off_s[C+1], scan_s[48], sidx_s[min(A, kLdsCopy)].
//
// A stable counting sort in blocks of one assignment per thread.  Inside a wavefront the lanes of one slot find
// each other from one ballot per bit of the slot id, so an assignment's rank among them is a population count;
// the wavefronts' counts per slot go through LDS, and the slots' offsets are one prefix sum.  Bound by the chain
// of LDS trips and barriers of one workgroup: 7.1 us at 1536 assignments on 48 slots, 95 us when every assignment
// counted the earlier ones of its slot one by one.
template <typename IdxPtr, typename TabPtr>
__device__ void block_post(IdxPtr idx, TabPtr slot_table, int A, int E, int C, int32_t *hist,
                           int32_t *slot_idx, int32_t *miss_list, int32_t *miss_count, int32_t *slot_count,
                           int32_t *slot_offset, int32_t *perm, int32_t *pos, int32_t *active_slots,
                           unsigned *n_active, unsigned *n_blocks, int block, lds_i32 *hist_s, lds_i32 *cnt_s, lds_i32 *off_s, lds_i32 *scan_s,
                           lds_i32 *sidx_s)
{
    static_assert(kMaxC <= kRouteThreads && kMaxC <= 1 << 10, "one thread per slot; ten bits of slot id");
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int nw = kRouteWaves;
    const unsigned long long below = (1ull << lane) - 1ull;
    if (hist)
        for (int e = tid; e < E; e += kRouteThreads) hist_s[e] = 0;
    for (int i = tid; i < nw * C; i += kRouteThreads) cnt_s[i] = 0;
    if (tid < C) off_s[tid] = 0;   // (assignments of each slot so far)
    __syncthreads();
    int running = 0;
    for (int base = 0; base < A; base += kRouteThreads) {
        const int a = base + tid;
        const bool valid = a < A;
        int c = -1;
        if (valid) {
            if (slot_table) {
                const int e = idx[a];
                const bool e_ok = (unsigned)e < (unsigned)E;
                if (hist && e_ok) __hip_atomic_fetch_add(&hist_s[e], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                c = e_ok ? slot_table[e] : -1;
            } else {
                c = slot_idx[a];
            }
            if ((unsigned)c >= (unsigned)C) c = -1;
            if (slot_table) slot_idx[a] = c;
        }
        const bool miss = valid && c < 0;
        const unsigned long long bal = __ballot(miss);
        // the lanes of this wavefront that name the same slot
        unsigned long long same = __ballot(c >= 0);
        for (int bit = 0; (C - 1) >> bit > 0; ++bit) {
            const unsigned long long on = __ballot((c >> bit) & 1);
            same &= ((c >> bit) & 1) ? on : ~on;
        }
        int r = __popcll(same & below);
        if (c >= 0 && r == 0) cnt_s[w * C + c] = __popcll(same);
        if (lane == 0) scan_s[w] = __popcll(bal);
        __syncthreads();
        // (only the wavefronts that hold an assignment have anything to add)
        const int left = A - base, nwv = left < kRouteThreads ? (left + kWave - 1) / kWave : nw;
        int wave_base = 0, total = 0;
        for (int i = 0; i < nwv; ++i) {
            const int s = scan_s[i];
            if (i < w) wave_base += s;
            total += s;
        }
        if (miss && miss_list) miss_list[running + wave_base + __popcll(bal & below)] = a;
        running += total;
        if (c >= 0) {
            r += off_s[c];
            for (int i = 0; i < w; ++i) r += cnt_s[i * C + c];
        }
        // rank and slot wait for the offsets: in LDS, or behind it in the words that they end up in
        if (valid) {
            if (a < kLdsCopy) sidx_s[a] = c >= 0 ? r << 10 | c : -1;
            else pos[a] = c >= 0 ? r : -1;
        }
        __syncthreads();
        if (tid < C) {
            int n = 0;
            for (int i = 0; i < nwv; ++i) {
                n += cnt_s[i * C + tid];
                cnt_s[i * C + tid] = 0;
            }
            off_s[tid] += n;
        }
        __syncthreads();
    }
    if (tid == 0 && miss_count) *miss_count = running;
    if (hist)
        for (int e = tid; e < E; e += kRouteThreads) hist[e] = hist_s[e];
    // offsets and active list: prefix sums of the counts and of the flag (count > 0) over the slots
    const int cntv = tid < C ? off_s[tid] : 0;
    int inc_o = cntv;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int v = __shfl_up(inc_o, d, kWave);
        if (lane >= d) inc_o += v;
    }
    const unsigned long long act = __ballot(cntv > 0);
    const unsigned blocks = wave_sum_u32((unsigned)(cntv + block - 1) >> (block == 32 ? 5 : 4));
    if (lane == kWave - 1) {
        scan_s[w] = (int)blocks;   // (the misses' counts are no longer needed)
        scan_s[16 + w] = inc_o;
        scan_s[32 + w] = __popcll(act);
    }
    __syncthreads();
    int base_o = 0, base_a = 0, tot_o = 0, tot_a = 0;
    for (int i = 0; i < (C + kWave - 1) / kWave; ++i) {
        const int vo = scan_s[16 + i], va = scan_s[32 + i];
        if (i < w) {
            base_o += vo;
            base_a += va;
        }
        tot_o += vo;
        tot_a += va;
    }
    if (tid < C) {
        const int off = base_o + inc_o - cntv;
        off_s[tid] = off;
        slot_offset[tid] = off;
        slot_count[tid] = cntv;
        if (cntv > 0) active_slots[base_a + __popcll(act & below)] = tid;
    }
    if (tid == 0) {
        slot_offset[C] = tot_o;
        *n_active = (unsigned)tot_a;
        int nb = 0;
        for (int i = 0; i < (C + kWave - 1) / kWave; ++i) nb += scan_s[i];
        *n_blocks = (unsigned)nb;
    }
    __syncthreads();
    // lists: assignment a goes to position off[slot] + (number of earlier assignments of that slot),
    // so the list of a slot holds its assignments in ascending flat id
    for (int a = tid; a < A; a += kRouteThreads) {
        int c, r;
        if (a < kLdsCopy) {
            const int v = sidx_s[a];
            c = v < 0 ? -1 : v & 1023;
            r = v >> 10;
        } else {
            r = pos[a];   // (written by this thread)
            c = r < 0 ? -1 : slot_idx[a];
        }
        if (c < 0) {
            pos[a] = -1;
            continue;
        }
        const int p = off_s[c] + r;
        perm[p] = a;
        pos[a] = p;
    }
}

// dynamic LDS: hist_s[E] tab_s[E] cnt_s[waves*C] off_s[C+1] scan_s[48] sidx_s[cap] idx_s[cap] lg_s[waves*E]
struct PostLds {
    lds_i32 *hist_s, *tab_s, *cnt_s, *off_s, *scan_s, *sidx_s, *idx_s;
    lds_f32 *lg_s;
};

__device__ inline PostLds carve_lds(int *dyn_, int E, int C, int A)
{
    const int cap = A < kLdsCopy ? A : kLdsCopy;
    lds_i32 *dyn = (lds_i32 *)dyn_;
    PostLds p;
    p.hist_s = dyn;
    p.tab_s = p.hist_s + E;
    p.cnt_s = p.tab_s + E;
    p.off_s = p.cnt_s + kRouteWaves * C;   // (counters of the general builder, or up to four mask words per slot)
    p.scan_s = p.off_s + C + 1;
    p.sidx_s = p.scan_s + 48;
    p.idx_s = p.sidx_s + cap;
    p.lg_s = (lds_f32 *)(dyn + ((2 * E + (kRouteWaves + 1) * C + 49 + 2 * cap + 3) & ~3));
    return p;
}

__host__ __device__ inline size_t post_lds_bytes(int E, int C, int A, bool with_topk)
{
    const int cap = A < kLdsCopy ? A : kLdsCopy;
    size_t n = (size_t)2 * E + (size_t)kRouteWaves * C + (C + 1) + 48 + 2 * cap;
    if (with_topk) n += (size_t)kRouteWaves * lg_stride(E) + 4;
    return n * sizeof(int);
}

constexpr int kSpinLimit = 1 << 20;   // polls of an entry in memory before a waiting workgroup gives up

// Small batches (T <= 128, one thread per assignment and per slot): the tokens of each slot as a
// bit mask of NW = ceil(T/32) words (a token names a slot at most once, the slot table being
// one-to-one), so counts, offsets and list positions are population counts.  Same outputs as
// block_post.
// PUBLISH: every word of the per-slot lists also goes, stamped with the call's number, into each of the
// kListReplicas copies behind r.lists_pub (entries no expert fills are stamped too, with -1, so that a
// reader can wait for all of them).
// What block_post_small found, in registers: thread tid < C holds slot tid's count, offset and place among the
// active slots (-1: no token); thread tid < T*k holds its assignment's slot and list position (-1: not
// resident); every thread holds the totals.
struct SmallLists {
    int count, offset, active_rank, n_active, n_listed, slot, pos;
};

// to_memory false: nothing is written to global memory (a workgroup that only wants the lists for itself).
// BLOCKS: also r.n_blocks (a template argument: the small batches' serial path has no use for it).
template <bool PUBLISH, bool BLOCKS = false>
__device__ __forceinline__ SmallLists block_post_small(lds_i32 *idx_s, lds_i32 *tab_s, int T, int kk, int E, int C, const RouteArgs &r,
                                 lds_i32 *hist_s, lds_i32 *mask_s, lds_i32 *scan_s, lds_i32 *off_s, unsigned tag,
                                 bool to_memory = true)
{
    auto publish = [&](int word, int value) {
        if (!PUBLISH) return;
        const unsigned long long e = ((unsigned long long)tag << 32) | (unsigned)value;
        const size_t stride = list_pub_entries(T, kk, C);
        for (int rep = 0; rep < kListReplicas; ++rep)
            __hip_atomic_store(r.lists_pub + rep * stride + word, e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
    const int A = T * kk, NW = (T + 31) >> 5;
    const bool valid = tid < A;
    const int tok = valid ? tid / kk : 0;
    int c = -1;
    if (valid) {
        const int e = idx_s[tid];
        __hip_atomic_fetch_add(&hist_s[e], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        c = tab_s[e];
        if ((unsigned)c >= (unsigned)C) c = -1;
        if (c >= 0)
            __hip_atomic_fetch_or(&mask_s[c * NW + (tok >> 5)], 1 << (tok & 31), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_WORKGROUP);
        if (to_memory) r.slot_idx[tid] = c;
    }
    const bool miss = valid && c < 0;
    const unsigned long long bal = __ballot(miss);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) scan_s[w] = __popcll(bal);
    __syncthreads();
    // slot `tid`: its token count; prefix sums of (count, count > 0) inside the wavefront, from ballots:
    // of the flag, and of each bit of the count (a count is at most T <= 128)
    int cntv = 0;
    if (tid < C)
        for (int wd = 0; wd < NW; ++wd) cntv += __popc((unsigned)mask_s[tid * NW + wd]);
    const unsigned long long upto = (2ull << lane) - 1ull;   // lanes 0..lane
    const int inc_a = __popcll(__ballot(cntv > 0) & upto);
    int inc_o = 0;
    for (int bit = 0; (1 << bit) <= T; ++bit) inc_o += __popcll(__ballot((cntv >> bit) & 1) & upto) << bit;
    const unsigned blocks = BLOCKS ? wave_sum_u32((unsigned)(cntv + stream_block(T) - 1) >> (T > 16 ? 5 : 4)) : 0u;
    if (lane == kWave - 1) {
        scan_s[16 + w] = inc_o;
        scan_s[32 + w] = BLOCKS ? inc_a | (int)blocks << 16 : inc_a;
    }
    // (only the wavefronts that hold an assignment or a slot have anything to add)
    const int nwv = ((A > C ? A : C) + kWave - 1) / kWave;
    {
        int wave_base = 0, total = 0;
        for (int i = 0; i < nwv; ++i) {
            const int v = scan_s[i];
            if (i < w) wave_base += v;
            total += v;
        }
        if (to_memory) {
            if (miss) r.miss_list[wave_base + before] = tid;
            if (tid == 0) *r.miss_count = total;
            if (tid < E) r.hist[tid] = hist_s[tid];
        }
    }
    __syncthreads();
    int base_o = 0, base_a = 0, tot_o = 0, tot_a = 0, tot_b = 0;
    for (int i = 0; i < nwv; ++i) {
        const int vo = scan_s[16 + i], vb = scan_s[32 + i], va = BLOCKS ? vb & 0xffff : vb;
        if (BLOCKS) tot_b += vb >> 16;
        if (i < w) {
            base_o += vo;
            base_a += va;
        }
        tot_o += vo;
        tot_a += va;
    }
    SmallLists out = {0, 0, -1, tot_a, tot_o, c, -1};
    if (tid < C) {
        const int off = base_o + inc_o - cntv, na = base_a + inc_a - (cntv > 0 ? 1 : 0);
        off_s[tid] = off;
        out.count = cntv;
        out.offset = off;
        out.active_rank = cntv > 0 ? na : -1;
        if (to_memory) {
            r.slot_count[tid] = cntv;
            r.slot_offset[tid] = off;
            if (cntv > 0) r.active_slots[na] = tid;
        }
        publish(1 + tid, cntv);
        publish(1 + C + tid, off);
        if (cntv > 0) publish(1 + 2 * C + na, tid);
        if (tid >= tot_a) publish(1 + 2 * C + tid, -1);
    }
    if (tid == 0) {
        if (to_memory) {
            r.slot_offset[C] = tot_o;
            *r.n_active = (unsigned)tot_a;
            if (BLOCKS) *r.n_blocks = (unsigned)tot_b;
        }
        publish(0, tot_a);
    }
    __syncthreads();
    // position of an assignment = offset of its slot + number of earlier tokens of that slot
    if (valid) {
        int p = -1;
        if (c >= 0) {
            p = off_s[c] + __popc((unsigned)mask_s[c * NW + (tok >> 5)] & ((1u << (tok & 31)) - 1u));
            for (int wd = 0; wd < (tok >> 5); ++wd) p += __popc((unsigned)mask_s[c * NW + wd]);
            if (to_memory) r.perm[p] = tid;
            publish(1 + 3 * C + p, tid);
        }
        if (to_memory) r.pos[tid] = p;
        out.pos = p;
        if (tid >= tot_o) publish(1 + 3 * C + tid, -1);
    }
    return out;
}

}  // namespace

}  // namespace moe
