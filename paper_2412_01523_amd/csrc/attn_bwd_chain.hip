// Backward of packed attention in one pass over the key tiles (D = 128): S and dP are formed once and dQ, dK and dV taken from them, where
// the two-kernel backward (attn_bwd.hip) forms them twice: five matrix products instead of seven.
//
// One work item = 128 keys of one (sequence, kv head), as there: dK^T and dV^T stay in registers while the query rows go by, 64 a
// step.  dQ of those rows is a sum over the key tiles, so it travels: the item of key tile b reads what tile b - 1 has left, adds its
// own dS K in fp32 and leaves it for tile b + 1; the last one to see the rows scales, rounds and writes dq.  The order of the
// additions is that of the keys, whoever runs when: results are bitwise reproducible, no float atomics, and dQ has the two kernels' bits where they cut no tile
// (dK and dV are summed from the last query rows to the first here).  A flag per (64 query rows,
// head) says how many key tiles have added.  Every item walks its query tiles from the last one down, so that the items of a sequence
// start together, each a step or two behind the one before, and with a mask the later, shorter walks end first.
// The rows in between (32 KB per step and item, read and written) stay in the L2 of the compute die that runs the neighbouring key tiles
// at that time: plain stores, loads that pass by the compute unit's own cache (sc1).  Measured on a buffer that a die's 32 compute units
// hand round: every such load sees the store, 12 TB/s read and as much written over the chip.  From die to die both go through
// memory (2.8 TB/s), so that only the last item of a bundle (see chain_take) stores its rows that way.
// What the hand-over relies on.  Within a die: a plain store that has been counted (vmcnt) is in the die's L2, and an sc1 load asks there; a
// wavefront that reads its own store back like that has to see it, and the L2 does not tell one unit's stores from another's.  From die to die: rows
// and flag are stored and loaded with sc1, which is what relaxed atomic accesses of agent scope are made of; such a load may not return an older copy
// that its die's L2 still holds (whoever waits for a flag of another die's would wait for good), so it does not matter which versions of
// a row a die has seen before.  The flag is stored when the rows have been counted.  Nobody reads rows of dQ in any other way, nor before the
// flag says that they are there: no load ahead of time, plain or not.
// What bounds it: on long sequences the matrix unit is busy for half of the cycles (counters: 49 %, short ones 26), and the chip is at 1.8 to 1.95 GHz
// (zero inputs: 2.3).  A workgroup of
// eight wavefronts has a compute unit to itself, two to a SIMD with 256 registers each.  While one of the two does matrix work alone
// (sums) the other forms S, dP and their exponentials (scores): wavefronts 0 .. 3 in this order, 4 .. 7 in the other.
// Of the rows' stores 24 % leave the L2 on long sequences all the same: what 32 workgroups two steps apart are busy with is as large as it.
// Backward, two kernels -> this, us: 8 heads, one sequence of 131 072 tokens 99 470 -> 88 610, 32 768 6 436 -> 5 530; 65 536 tokens in sequences of 4 096
// 1 853 -> 1 659, 2 048 1 089 -> 982, 1 024 622 -> 615; 49 152 tokens, up to 1 024 a sequence 393 -> 380; a 64K-token long-tail batch 1 305 -> 1 228;
// 262 144 tokens, 16 heads on 2 120 650 -> 108 680.
// Tried on the way: both wavefronts of a SIMD in the same phase, two barriers a step (as fast as two kernels); the exponentials between the
// sums' matrix instructions of the same wavefront (56 registers too many).
#include <type_traits>

#include "attn_common.h"

namespace flexsp {
namespace {

// LDS fragments are read this many matrix instructions ahead (the file is compiled in source order); 4 takes 2 % longer, 2 the same
constexpr int kReadAhead = 3;
constexpr int kChainThreads = 512;
constexpr int kDeltaRows = kThreads / 64 * 32;

// ------------------------------------------------------------------------------ delta
// -delta = -(dO . O) and the base-2 log-sum-exp of every row, and a clear dealer and flags for the launch behind it.  One wavefront: 32
// rows of one head, read as whole rows and summed in the order of the dQ kernel (attn_bwd.hip): half a row's head dims in turn by a lane, then
// the other half's sum, so that dQ has the bits it has there.  Bound by reading O and dO: 65 536 tokens, 8 heads 61 us between events (53
// with pieces summed by whichever lanes read them, and rounded differently).  (The key tiles all need delta, none before the
// others, so no item of theirs can form it for the rest.)
__global__ __launch_bounds__(kThreads) void attn_bwd_delta_kernel(const AttnArgs)
{
    constexpr int D = 128, KS = D / 16;
    typedef LdsTile<D> L;
    __shared__ __attribute__((aligned(1024))) char smem[kThreads / 64 * 32 * L::ROWB];
    KernArgs &a = kernel_args();
    const int tid = thread_id(), wg = workgroup_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int h = wg % a.Hq, t0 = wg / a.Hq * kDeltaRows + wave * 32;
    LaneOffsets<D> lo;
    lo.init(lane);
    RowBlock<D> orows, grows;
    orows.load(a.o + (int64_t)h * a.o_sh, a.o_st, t0, a.T - 1, lane);
    grows.load(a.dO + (int64_t)h * a.do_sh, a.do_st, t0, a.T - 1, lane);
    char *const region = smem + wave * (32 * L::ROWB);
    bf16x8 of[KS], gf[KS];
    orows.fragments(region, 0, lo, of, lane);
    grows.fragments(region, 0, lo, gf, lane);
    float d = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ks++) {
        Frag8 fg, fo;
        fg.v = gf[ks];
        fo.v = of[ks];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t gw = fg.u[i], ow = fo.u[i];
            d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, gw), __builtin_bit_cast(bf16x2, ow), d, false);
        }
    }
    d = halves_sum(d);
    const int64_t at = (int64_t)h * a.T + t0 + lane;
    if (lane < 32 && t0 + lane < a.T) {
        a.delta_out[at] = -d;
        a.lse_out[at] = a.lse_in[at] * 1.4426950408889634f;
    }
    for (int i = wg * kThreads + tid; i < a.chain_flags; i += a.grid * kThreads) a.pq.split_flags[i] = 0;
    if (wg == 0 && tid <= kChainDies) *(unsigned long long *)(a.pq.counters + tid * kCounterStride) = 0;
}

// ------------------------------------------------------------------------------ work
// The workgroups' side of chain_take.
struct ChainDealer {
    const int32_t *offsets;
    uint32_t *next;            // bundles taken
    unsigned long long *word;  // this die's
    typedef volatile __attribute__((address_space(3))) int Word;
    Word *slot;
    int bundles, wave, lane;
    unsigned long long pending;

    __device__ __forceinline__ unsigned long long draw()
    {
        unsigned long long w = 0;
        if (lane == 0) w = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return w;
    }
    __device__ __forceinline__ unsigned long long look() { return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ void put(unsigned long long w)
    {
        if (lane == 0) __hip_atomic_store(word, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t bundle()
    {
        uint32_t b = 0;
        if (lane == 0) b = __hip_atomic_fetch_add(next, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return __builtin_amdgcn_readfirstlane(b);
    }
    __device__ __forceinline__ uint32_t low(unsigned long long w) { return __builtin_amdgcn_readfirstlane((uint32_t)w); }
    __device__ __forceinline__ uint32_t high(unsigned long long w) { return __builtin_amdgcn_readfirstlane((uint32_t)(w >> 32)); }
    __device__ __forceinline__ void rest() { __builtin_amdgcn_s_sleep(1); }
    __device__ __forceinline__ int take(unsigned long long w)  // wavefront 0
    {
        return __builtin_amdgcn_readfirstlane(chain_take(*this, w, offsets, bundles));
    }
    __device__ __forceinline__ int publish(int idx)
    {
        if (wave == 0 && lane == 0) *slot = idx;
        __builtin_amdgcn_s_waitcnt(0xC07F);
        __builtin_amdgcn_s_barrier();
        return __builtin_amdgcn_readfirstlane(*slot);
    }
    __device__ __forceinline__ int first(KernQueues &pq, int &lds_word, int wave_, int lane_)
    {
        int die;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(die));
        offsets = pq.offsets;
        bundles = pq.nq;
        next = (uint32_t *)pq.counters;
        word = (unsigned long long *)(pq.counters + (1 + (die & (kChainDies - 1))) * kCounterStride);
        slot = (Word *)(uintptr_t)(uint32_t)(uintptr_t)&lds_word;
        wave = wave_;
        lane = lane_;
        pending = 0;
        return publish(wave == 0 ? take(draw()) : -1);
    }
    __device__ __forceinline__ void prefetch()
    {
        if (wave == 0) pending = draw();
    }
    __device__ __forceinline__ int advance() { return publish(wave == 0 ? take(pending) : -1); }
};

// A flag into LDS, past the compute unit's own cache.
__device__ __forceinline__ void flag_to_lds(const int32_t *g, void *lds)
{
    const uint32_t dst = (uint32_t)(uintptr_t)lds;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off sc1" ::"v"(g), "s"(dst) : "memory");
}

// As global_to_lds16 with a base in scalar registers.  A scalar register that a vector instruction has written (v_readlane: this kernel's scalars do not all
// fit, and wait in lanes of a vector register) may be a memory instruction's address five wait states later at the earliest; the hardware does
// not wait, and the compiler does not count for an inline assembly statement.  So the statement counts itself (the write of m0 is one of
// them).
__device__ __forceinline__ void scalar_to_lds16(const void *base, uint32_t lane_off, void *lds)
{
    const uint32_t dst = (uint32_t)(uintptr_t)lds;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(dst) : "memory");
}
// A wavefront's share of two tiles in one statement, which counts once: `a0`, `a1` of `a` to lds and GAP bytes behind, `b0`, `b1` of `b` to 2 and 3 GAP
// behind.  The wavefronts that copy right behind the barrier hold everybody up meanwhile: one sequence of 131 072 tokens, 8 heads 90 960 -> 89 130 us
// against four statements, shorter ones the same.
template <int GAP>
__device__ __forceinline__ void scalar_to_lds16(const void *a, uint32_t a0, uint32_t a1, const void *b, uint32_t b0, uint32_t b1, void *lds)
{
    const uint32_t dst = (uint32_t)(uintptr_t)lds;
    asm volatile("s_mov_b32 m0, %6\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %4\n\t"
                 "s_add_u32 m0, %6, %7\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %4\n\t"
                 "s_add_u32 m0, %6, %8\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %5\n\t"
                 "s_add_u32 m0, %6, %9\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, %5" ::"v"(a0), "v"(a1), "v"(b0), "v"(b1), "s"(a), "s"(b), "s"(dst),
                 "n"(GAP), "n"(2 * GAP), "n"(3 * GAP) : "memory", "scc");
}
__device__ __forceinline__ void scalar_to_lds4(const void *base, uint32_t lane_off, void *lds)
{
    const uint32_t dst = (uint32_t)(uintptr_t)lds;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(base), "s"(dst) : "memory");
}

__global__ __launch_bounds__(kChainThreads, 2) void attn_bwd_chain_kernel(const AttnArgs)
{
    constexpr int D = 128, T = kChainThreads;
    typedef LdsTile<D> L;
    typedef LdsTile<64> L64;
    constexpr int KS = D / 16, DB = D / 32, BQ = kDkvBq;
    constexpr int QTILE = BQ * L::ROWB;
    constexpr int STEP = 2 * QTILE + 512;      // Q | dO | lse2[64] -delta[64]
    constexpr int NB = 3;
    constexpr int DS = NB * STEP;              // two of: dS, [key][64 queries]
    constexpr int DSB = kChainBk * L64::ROWB;
    constexpr int EX = DS + 2 * DSB;           // two of: P of query block 1, a fragment set per key block
    constexpr int EXB = 4 * 2048;
    constexpr int FLAG = EX + 2 * EXB, NOBODY = FLAG + 256;
    constexpr int ZERO = NOBODY + 256;         // 32 rows of zeros, read in place of rows that a key block's P and dS have no terms of
    __shared__ __attribute__((aligned(1024))) char smem[ZERO + 32 * L::ROWB];
    __shared__ int deal_word;
    KernArgs &args = kernel_args();

    const int tid = thread_id();
    const int lane0 = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = wave & 3;
    const bool ahead = wave < 4;  // dK and query block 1; the others: dV and query block 0
    static_assert(32 * L::ROWB == T * 16, "a piece each");
    *(u32x4 *)(smem + ZERO + tid * 16) = u32x4{0, 0, 0, 0};  // (visible behind the dealer's barrier)
    ChainDealer deal;

    for (int item = deal.first(args.pq, deal_word, wave, lane0); item >= 0; item = deal.advance()) {
        KernArgs &a = fresh(args);
        const flexsp_item it = load_item(a.pq.items, item);
        const int s = it.seq_len, g = it.head, b = it.tile, kv0 = b * kChainBk;
        const int64_t tok0 = it.seq_start;
        const bool causal = a.causal != 0, far = it.parts != 0;  // far: the next block's bundle may be another die's
        const int nt = (s + BQ - 1) / BQ, t_first = causal ? kv0 / BQ : 0, G = a.G;
        const int n = (nt - t_first) * G;
        const int last_below = causal ? t_first + kChainBk / BQ : kv0 + kChainBk >= s ? nt : 0;  // tiles below this: nobody adds to them after this block
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        lane &= 63;
        const int wk_lo = kv0 + kb * 32;
        const int clear_from = wk_lo + 32 > s ? 0x7fffffff : causal ? wk_lo + 31 : 0;  // blocks of queries from here on, up to the end, have nothing to mask

        const int seen_from = causal ? wk_lo - 31 : 0;  // no row of a block of queries below this sees a key of the wavefront's
        // The step fetched next: its tiles' first rows, its statistics, the copies of a lane's rows
        const char *q_f = (const char *)(a.q + (tok0 + (int64_t)(nt - 1) * BQ) * a.q_st + (int64_t)g * a.G * a.q_sh);
        const char *g_f = (const char *)(a.dO + (tok0 + (int64_t)(nt - 1) * BQ) * a.do_st + (int64_t)g * a.G * a.do_sh);
        const char *s_f = (const char *)((wave == 5 ? a.delta_in : a.lse_in) + (int64_t)g * a.G * a.T + tok0 + (nt - 1) * BQ);
        int t_f = nt - 1, h_f = 0, base_f = 0;
        int rows_f;  // rows of that tile
        uint32_t oq0, oq1, og0, og1;
        auto lane_rows = [&](int rows) {  // for a tile of that many rows: lanes of those past the end repeat the last one
            int l = lane;
            asm volatile("" : "+v"(l));
            const int row = wave * 4 + (l >> 4), col = ((l & 15) ^ L::sw(row)) << 4;
            oq0 = min(row, rows - 1) * (uint32_t)a.q_st * 2u + col;
            oq1 = min(row + 32, rows - 1) * (uint32_t)a.q_st * 2u + col;
            og0 = min(row, rows - 1) * (uint32_t)a.do_st * 2u + col;
            og1 = min(row + 32, rows - 1) * (uint32_t)a.do_st * 2u + col;
            asm volatile("" : "+v"(oq0), "+v"(oq1), "+v"(og0), "+v"(og1));  // (multiplied in 64 bits: a register each, not two)
            rows_f = rows;
        };
        lane_rows(min(BQ, s - (nt - 1) * BQ));
        auto copy = [&](int i) {
            char *const dst = smem + base_f + (i >> 1) * QTILE + (i & 1) * (QTILE / 2) + wave * 1024;
            scalar_to_lds16(i < 2 ? q_f : g_f, i == 0 ? oq0 : i == 1 ? oq1 : i == 2 ? og0 : og1, dst);
        };
        // (the statistics by two of wavefronts 4 .. 7, whose copies have a whole window's time)
        auto copy_stats = [&]() {
            if (wave == 4 || wave == 5) {
                int l = lane;
                asm volatile("" : "+v"(l));
                scalar_to_lds4(s_f, min(l, rows_f - 1) * 4, smem + base_f + 2 * QTILE + wave * 256 - 1024);
            }
        };
        auto copy_all = [&]() {
            copy_stats();
            scalar_to_lds16<QTILE / 2>(q_f, oq0, oq1, g_f, og0, og1, smem + base_f + wave * 1024);
        };
        auto copied = [&]() {  // (the heads of a tile one after the other, then the tile in front)
            base_f = base_f == (NB - 1) * STEP ? 0 : base_f + STEP;
            q_f += (int64_t)a.q_sh * 2;
            g_f += (int64_t)a.do_sh * 2;
            s_f += (int64_t)a.T * 4;
            if (++h_f == G) {
                h_f = 0;
                if (t_f == nt - 1) lane_rows(BQ);
                t_f--;
                q_f -= ((int64_t)G * a.q_sh + (int64_t)BQ * a.q_st) * 2;
                g_f -= ((int64_t)G * a.do_sh + (int64_t)BQ * a.do_st) * 2;
                s_f -= ((int64_t)G * a.T + BQ) * 4;
            }
        };
        // K and V pass through the second and the third step buffer
        load_tile_async<D, kChainBk, T>(smem + STEP, a.k + tok0 * a.k_st + (int64_t)g * a.k_sh, a.k_st, kv0, s - 1, wave, lane);
        load_tile_async<D, kChainBk, T>(smem + 2 * STEP, a.v + tok0 * a.v_st + (int64_t)g * a.v_sh, a.v_st, kv0, s - 1, wave, lane);
        copy_all();
        copied();
        wait_vmem();
        __syncthreads();

        auto role = [&](auto aheadc) {
            constexpr bool AHEAD = decltype(aheadc)::value;
            constexpr int j = AHEAD ? 1 : 0;
            // lane offsets; the other fragments lie at an exclusive-or (the swizzle works on the same bits)
            int nat0, tr0, dtr0, dst0;
            {
                const int r = lane & 31, hl = lane >> 5, i = lane & 15, gg = lane >> 4, cl = 2 * (gg & 1) + ((i & 3) >> 1), row = 4 * hl + (i >> 2);
                nat0 = r * L::ROWB + ((hl ^ L::sw(r)) << 4);
                tr0 = row * L::ROWB + ((cl ^ L::sw(row)) << 4) + (i & 1) * 8;
                dtr0 = DS + row * L64::ROWB + (((4 * j + cl) ^ L64::sw(row)) << 4) + (i & 1) * 8;
                dst0 = DS + (kb * 32 + r) * L64::ROWB + ((L64::sw(r) << 4) | (8 * hl));  // this lane's key row of dS
            }
            // transpose reads: the second four rows lie eight rows below the first, where the swizzle differs in one bit
            auto tr128 = [&](int off, int at) { return lds_tr(smem, off + at, (off ^ 32) + at + 8 * L::ROWB); };
            auto tr64 = [&](int off, int at) { return lds_tr(smem, off + at, (off ^ 32) + at + 8 * L64::ROWB); };
            // kf, vf: B operands of S and dP; kt: K^T of the head-dim block whose dQ this wavefront adds up
            bf16x8 kf[KS], vf[KS], kt[8];
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                kf[ks] = lds_nat(smem + STEP + kb * 32 * L::ROWB, nat0 ^ (ks << 5));
                vf[ks] = lds_nat(smem + 2 * STEP + kb * 32 * L::ROWB, nat0 ^ (ks << 5));
            }
#pragma unroll
            for (int i = 0; i < 8; i++) kt[i] = tr128(tr0 ^ (kb << 6), STEP + i * 16 * L::ROWB);
            nat0 += j * 32 * L::ROWB;
            tr0 += AHEAD ? 0 : QTILE;  // dK from Q, dV from dO
            f32x16 accT[DB];
#pragma unroll
            for (int d = 0; d < DB; d++)
#pragma unroll
                for (int i = 0; i < 16; i++) accT[d][i] = 0.f;
            uint32_t mine[8];  // !AHEAD: P of query block 0
            f32x16 dq;         // a block of dQ

            // a step: tile, head, place among the flags, step buffer, exchange buffer
            int t_x = nt - 1, h_x = g * a.G, i_x = it.slot * a.Hq + h_x * nt + t_x, b_x = 0, e_x = 0;
            int t_y = t_x, h_y = h_x, i_y = i_x, b_y = 0, e_y = 0;
            auto next_x = [&]() {
                b_x = b_x == (NB - 1) * STEP ? 0 : b_x + STEP;
                e_x ^= 1;
                i_x += nt;
                if (++h_x == (g + 1) * G) {
                    h_x = g * G;
                    i_x -= G * nt + 1;
                    t_x--;
                }
            };
            auto same = [&]() { t_y = t_x, h_y = h_x, i_y = i_x, b_y = b_x, e_y = e_x; };
            int pub = -1;  // flag of the tile added to last: raised once its rows are in memory

            auto raise = [&](int32_t *flags) {
                if (pub < 0 || lane != 0) return;
                if (far)
                    __hip_atomic_store(flags + pub, b + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else
                    __hip_atomic_store(flags + pub, b + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            // Window w begins: step w's tile has landed, the fragments of step w - 1 (the y step) are visible.
            auto window = [&](int w) {
                wait_vmem();
                if (AHEAD && wave == 0 && b > 0 && w > 0) {
                    int seen = *(ChainDealer::Word *)(uintptr_t)(uint32_t)(uintptr_t)(smem + FLAG);
                    seen = __builtin_amdgcn_readfirstlane(seen);
                    while (seen < b) {
                        __builtin_amdgcn_s_sleep(1);
                        seen = __hip_atomic_load(a.pq.split_flags + i_y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        seen = __builtin_amdgcn_readfirstlane(seen);
                    }
                }
                __syncthreads();
                if (AHEAD && wave == 0) {
                    raise(a.pq.split_flags);
                    if (b > 0 && w < n) flag_to_lds(a.pq.split_flags + i_x, smem + FLAG);
                }
            };
            // The first block of a bundle would meet every tile in memory, and the others keep its pace.  So the n-th block after
            // it touches the n-th eighth of a tile's lines (Q, dO) before it gets there.  (Not the lines of dQ that another bundle has added
            // to: whether that has added for the last time is what the flag says, and nobody reads a row of dQ before the flag.)
            const int nth = b - it.step_begin, reach = (2 * nth + 5) / G + 1;  // in tiles
            auto touch = [&]() {
                const int t = t_x - reach;
                if (nth < 1 || nth > 8 || t < (causal ? it.step_begin * (kChainBk / BQ) : 0)) return;
                int l = lane;
                asm volatile("" : "+v"(l));
                const bool is_q = nth <= 4;
                const int64_t row = tok0 + t * BQ + (nth - 1 & 3) * 16 + (l >> 2);
                global_to_lds4((const char *)((is_q ? a.q : a.dO) + row * (is_q ? a.q_st : a.do_st) + (int64_t)h_x * (is_q ? a.q_sh : a.do_sh)) + (l & 3) * 64, smem + NOBODY);
            };
            auto ask = [&]() {
                int l = lane;
                asm volatile("" : "+v"(l));
                const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc((void *)(a.pq.split_scratch + (int64_t)i_y * (int64_t)kChainTileBytes), 0, b > 0 ? (int)kChainTileBytes : 0, 0x00020000);
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(rows, l * 16, wave * 4096 + i * 1024, 16);
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        const uint32_t x = w[e];
                        dq[4 * i + e] = __builtin_bit_cast(float, x);
                    }
                }
            };
            // K^T's fragments whose keys no row of query block j sees any more, from tile t down: cleared, dS is zero for them but K need not be finite.
            // (Between two steps: the same in front of the sums took 2 to 3 % longer.)
            auto trim = [&](int t) {
                if (causal && t <= t_first + 1) {
                    if (!AHEAD) kt[6] = kt[7] = bf16x8{};
                    if (t == t_first) {
#pragma unroll
                        for (int i = AHEAD ? 4 : 2; i < (AHEAD ? 8 : 6); i++) kt[i] = bf16x8{};
                    }
                }
            };
            // S, dP, P and dS of query block j
            auto scores = [&](const bool more) {
                const int my_lo = t_x * BQ + j * 32;
                int l = lane, nat = nat0 + b_x, dst = dst0 + e_x * DSB;
                asm volatile("" : "+v"(l), "+v"(nat), "+v"(dst));
                const int st = (l >> 5) * 16 + (b_x + 2 * QTILE + j * 128);  // row statistics of this lane's rows
                char *const slot = smem + EX + e_x * EXB + kb * 2048 + l * 16;
                const bool clear = my_lo >= clear_from && my_lo + 32 <= s;
                if (clear || !(my_lo >= s || wk_lo >= s || (causal && my_lo + 31 < wk_lo))) {
                    f32x16 sacc, pacc;
#pragma unroll
                    for (int i4 = 0; i4 < 4; i4++) {
                        const f32x4 d4 = *(const f32x4 *)(smem + st + 256 + 32 * i4);
#pragma unroll
                        for (int e = 0; e < 4; e++) pacc[4 * i4 + e] = d4[e];
                    }
                    constexpr int AH = kReadAhead, N = 2 * KS;
                    bf16x8 fr[N];
                    f32x4 l4[4];
                    auto rd = [&](int i) { return lds_nat(smem, ((i & 1) ? QTILE : 0) + (nat ^ ((i >> 1) << 5))); };
#pragma unroll
                    for (int i = 0; i < AH; i++) fr[i] = rd(i);
#pragma unroll
                    for (int i = 0; i < N; i++) {
                        if (i + AH < N) fr[i + AH] = rd(i + AH);
                        if (i & 1)
                            pacc = mfma32(fr[i], vf[i >> 1], pacc);
                        else
                            sacc = mfma32(fr[i], kf[i >> 1], i ? sacc : f32x16{});
                        if (AHEAD && i % 4 == 2 && more) copy(i / 4);
                        if (i >= N - 4) l4[i - (N - 4)] = *(const f32x4 *)(smem + st + 32 * (i - (N - 4)));
                    }
                    if (AHEAD) ask();
                    auto probs = [&](auto maskc) {
                        constexpr bool MASK = decltype(maskc)::value;
                        uint32_t pp[8];
#pragma unroll
                        for (int i4 = 0; i4 < 4; i4++) {
                            float p[4], ds[4];
#pragma unroll
                            for (int e = 0; e < 4; e++) {
                                p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[4 * i4 + e], a.scale_l2, -l4[i4][e]));
                                if (MASK) {
                                    const int qr = my_lo + 8 * i4 + 4 * (l >> 5) + e, kvrow = wk_lo + (l & 31);
                                    p[e] = ((causal && qr < kvrow) || qr >= s || kvrow >= s) ? 0.f : p[e];
                                }
                                ds[e] = p[e] * pacc[4 * i4 + e];
                            }
                            pp[2 * i4] = pack_bf16x2(p[0], p[1]);
                            pp[2 * i4 + 1] = pack_bf16x2(p[2], p[3]);
                            *(u32x2 *)(smem + (dst ^ ((4 * j + i4) << 4))) = u32x2{pack_bf16x2(ds[0], ds[1]), pack_bf16x2(ds[2], ds[3])};
                            if (AHEAD) {
                                if (i4 & 1) *(u32x4 *)(slot + (i4 >> 1) * 1024) = u32x4{pp[2 * i4 - 2], pp[2 * i4 - 1], pp[2 * i4], pp[2 * i4 + 1]};
                            } else {
                                mine[2 * i4] = pp[2 * i4];
                                mine[2 * i4 + 1] = pp[2 * i4 + 1];
                            }
                        }
                    };
                    if (clear)
                        probs(std::false_type{});
                    else
                        probs(std::true_type{});
                } else {
                    if (AHEAD) ask();
#pragma unroll
                    for (int i4 = 0; i4 < 4; i4++) *(u32x2 *)(smem + (dst ^ ((4 * j + i4) << 4))) = u32x2{0, 0};
                    if (AHEAD) {
                        *(u32x4 *)slot = u32x4{0, 0, 0, 0};
                        *(u32x4 *)(slot + 1024) = u32x4{0, 0, 0, 0};
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; i++) mine[i] = 0;
                    }
                    if (AHEAD && more) {
                        copy(0);
                        copy(1);
                        copy(2);
                        copy(3);
                    }
                }
                if (AHEAD) copied();
            };
            // dQ's block, then dV or dK
            auto sums = [&]() {
                const bool last = t_y < last_below;
                // (zero times infinity is none: rows of Q and dO that no key of the block sees are read from the zeros)
                auto from = [&](int qb) {
                    const int lo = t_y * BQ + qb * 32;
                    return (qb && lo >= s) || lo < seen_from ? ZERO - (AHEAD ? 0 : QTILE) - qb * 32 * L::ROWB : b_y;
                };
                const int shift = from(1) - from(0);
                int l = lane, d0 = dtr0 + e_y * DSB, t0 = tr0 + from(0), dst = dst0 + e_y * DSB;
                asm volatile("" : "+v"(l), "+v"(d0), "+v"(t0), "+v"(dst));
                int ta[DB], tb[DB];  // a head-dim block's transpose reads (tr128), for query block 1 as for 0 but on the diagonal and in half a tile
#pragma unroll
                for (int d = 0; d < DB; d++) ta[d] = t0 ^ (d << 6), tb[d] = (ta[d] ^ 32) + 8 * L::ROWB;
                // B operands of a query block's sums
                auto operands = [&](int qb, Frag8 (&f)[2]) {
                    if (AHEAD) {
#pragma unroll
                        for (int hf = 0; hf < 2; hf++) {
                            const u32x2 x = *(const u32x2 *)(smem + (dst ^ ((4 * qb + 2 * hf) << 4)));
                            const u32x2 y = *(const u32x2 *)(smem + (dst ^ ((4 * qb + 2 * hf + 1) << 4)));
                            f[hf].u = u32x4{x[0], x[1], y[0], y[1]};
                        }
                    } else if (qb == 0) {
                        f[0].u = u32x4{mine[0], mine[1], mine[2], mine[3]};
                        f[1].u = u32x4{mine[4], mine[5], mine[6], mine[7]};
                    } else {
                        const char *slot = smem + EX + e_y * EXB + kb * 2048 + l * 16;
                        f[0].u = *(const u32x4 *)(slot);
                        f[1].u = *(const u32x4 *)(slot + 1024);
                    }
                };
                // Twenty-four matrix instructions: the sums' sixteen, dQ's eight in turn with those from the fifth on.  On the diagonal those of
                // blocks above it multiply zeros by zeros: each under a condition of its own takes 15 % longer altogether, a second form of this for
                // such tiles 4 %.
                constexpr int AH = kReadAhead, LEAD = 4, N = 24;
                bf16x8 fr[N];
                Frag8 f[2];
                auto is_dq = [](int i) { return i >= LEAD && i < LEAD + 16 && !((i - LEAD) & 1); };
                auto sum_no = [](int i) { return i < LEAD ? i : i < LEAD + 16 ? LEAD + ((i - LEAD) >> 1) : i - 8; };
                auto rd = [&](int i) {
                    if (is_dq(i)) return tr64(d0, ((i - LEAD) >> 1) * 16 * L64::ROWB);
                    const int x = sum_no(i);
                    if (x == 8 && __builtin_expect(shift != 0, 0)) {
#pragma unroll
                        for (int d = 0; d < DB; d++) ta[d] += shift, tb[d] += shift;
                    }
                    const int off = ((x >> 3) * 32 + (x & 7) / DB * 16) * L::ROWB;
                    return lds_tr(smem, ta[x % DB] + off, tb[x % DB] + off);
                };
                operands(0, f);
#pragma unroll
                for (int i = 0; i < AH; i++) fr[i] = rd(i);
#pragma unroll
                for (int i = 0; i < N; i++) {
                    if (i + AH < N) fr[i + AH] = rd(i + AH);
                    if (is_dq(i)) {
                        dq = mfma32(kt[(i - LEAD) >> 1], fr[i], dq);
                    } else {
                        const int x = sum_no(i);
                        accT[x % DB] = mfma32(fr[i], f[(x & 7) / DB].v, accT[x % DB]);
                        if (x == 7) operands(1, f);
                    }
                }
                if (!last) {
                    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc((void *)(a.pq.split_scratch + (int64_t)i_y * (int64_t)kChainTileBytes), 0, (int)kChainTileBytes, 0x00020000);
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const f32x4 w = {dq[4 * i], dq[4 * i + 1], dq[4 * i + 2], dq[4 * i + 3]};
                        if (far)
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), rows, l * 16, wave * 4096 + i * 1024, 16);
                        else
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, w), rows, l * 16, wave * 4096 + i * 1024, 0);
                    }
                } else {
                    const int qr = t_y * BQ + j * 32 + (l & 31);
                    const int64_t at = (tok0 + qr) * a.dq_st + (int64_t)h_y * a.dq_sh + kb * 32;
                    const float mul = a.scale;
                    if (a.grad_f32) {
                        if (qr < s)
#pragma unroll
                            for (int i = 0; i < 4; i++) *(f32x4 *)((float *)a.dq + at + 8 * i + 4 * (l >> 5)) = f32x4{dq[4 * i] * mul, dq[4 * i + 1] * mul, dq[4 * i + 2] * mul, dq[4 * i + 3] * mul};
                    } else {
                        // (the half-waves hold four head dims of eight each: exchanged, a lane has all eight of one half's)
#pragma unroll
                        for (int i = 0; i < 4; i += 2) {
                            uint32_t x[2], y[2];
#pragma unroll
                            for (int e = 0; e < 2; e++) {
                                const uint32_t lo = pack_bf16x2(dq[4 * i + 2 * e] * mul, dq[4 * i + 2 * e + 1] * mul), hi = pack_bf16x2(dq[4 * i + 4 + 2 * e] * mul, dq[4 * i + 5 + 2 * e] * mul);
                                const auto both = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
                                x[e] = both[0];
                                y[e] = both[1];
                            }
                            if (qr < s) *(u32x4 *)((uint16_t *)a.dq + at + 8 * i + 8 * (l >> 5)) = u32x4{x[0], x[1], y[0], y[1]};
                        }
                    }
                }
                pub = last ? -1 : i_y;
            };
            if (!AHEAD) {
                window(0);
                if (n > 1) copy_all();
                copied();
            }
            for (int w = 0; w < n; w++) {
                asm volatile("" : "=v"(dq));  // (nothing passes from one round of this loop to the next in these)
#pragma unroll
                for (int i = 0; i < 8; i++) asm volatile("" : "=v"(mine[i]));
                if (AHEAD) window(w);
                if (!AHEAD && wave == 7) touch();
                if (!AHEAD) trim(t_x);
                scores(w + 1 < n);
                if (!AHEAD) {
                    same();
                    window(w + 1);
                    // (first of all: asked for in scores, their time beyond that is all waiting for the block that meets them in memory; and the
                    // block in front is everybody's pace: 2 to 4 %)
                    if (w + 2 < n) copy_all();
                    copied();
                    ask();
                }
                if (!AHEAD || w > 0) sums();
                if (AHEAD) {
                    same();
                    trim(t_x);
                }
                next_x();
            }
            if (AHEAD) {
                window(n);
                ask();
                sums();
            }
            KernArgs &e = fresh(args);
            deal.prefetch();
            wait_vmem();
            __syncthreads();  // every wavefront's last rows of dQ are in memory, and nobody reads the tiles any more
            if (AHEAD && wave == 0) raise(e.pq.split_flags);

            char *const out = (char *)(AHEAD ? e.dk : e.dv);
            const int64_t ost = AHEAD ? e.dk_st : e.dv_st, osh = AHEAD ? e.dk_sh : e.dv_sh;
            const float mul = AHEAD ? e.scale : 1.0f;
            if (wk_lo >= s) return;
            char *const stage = smem + wave * (32 * L::ROWB);
            if (e.grad_f32) {
                RowsF32<DB> f;
                f.store(stage, (float *)out + (tok0 + wk_lo) * ost + (int64_t)g * osh, ost, min(32, s - wk_lo), accT, mul, lane);
            } else {
                store_rowT_bf16_lds<DB>(stage, (uint16_t *)out + (tok0 + wk_lo) * ost + (int64_t)g * osh, ost, min(32, s - wk_lo), accT, mul, lane);
            }
        };
        if (ahead)
            role(std::true_type{});
        else
            role(std::false_type{});
    }
}

}  // namespace

hipError_t launch_attn_bwd_delta(const AttnArgs &a, hipStream_t s)
{
    launch(attn_bwd_delta_kernel, a, (int)((a.T + kDeltaRows - 1) / kDeltaRows) * a.Hq, s);
    return hipGetLastError();
}

hipError_t launch_attn_bwd_chain(const AttnArgs &a, int grid, hipStream_t s)
{
    AttnArgs with_grid = a;
    with_grid.grid = grid;
    hipLaunchKernelGGL(attn_bwd_chain_kernel, dim3(grid), dim3(kChainThreads), 0, s, with_grid);
    return hipGetLastError();
}

}  // namespace flexsp
