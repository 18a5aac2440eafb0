// Step loops that keep a class's gains in registers (gfx950), one workgroup per class: the graph-cut function and the
// incremental-gain route, for classes of up to a few thousand samples.
//
// What bounds these loops is latency: a step is a chain of a scan, a reduction, a trip to memory for row v* of S and, on
// the incremental route, a second trip for the rows whose coverage changed.  The loops of incremental_kernels.hip walk
// that chain once per step with the gains in L2.  Here
//   - the gains of all blocks sit in the registers of the workgroup (n x K doubles: 160 KB for 5000 samples and four
//     blocks, of the 512 KB a compute unit has), so the scan is arithmetic;
//   - the block state (f, room left) sits in the lanes of every wave, so choosing the block is one wave reduction;
//   - picks run ahead of updates.  Taking v* into block k changes the gains of block k only (and strikes v* out
//     everywhere), so the next block's argmax can be taken while row v* is still on its way, unless that block is k again.
// The order of the steps, every sum and every tie are those of the other loops: the results are the same bits.
// Graph cut, one class, us per step before -> after: 250 samples and 2 blocks 2.25 -> 0.90, 1000 / 8 2.28 -> 0.98,
// 3000 / 8 2.54 -> 0.99, 5000 / 4 3.14 -> 1.14; ten classes of 5000 with 4 blocks, whole call 19.8 -> 8.0 ms.  What is left
// of a step is about 350 instructions of one wave after the other's result, and the barrier.
//
// Layout: wave w owns the samples [128 Q w, 128 Q (w + 1)), in Q pieces of 128; lane l holds samples 2 l and 2 l + 1 of
// each piece (8-byte loads, 512 contiguous bytes per wave).
// Included by rcd_lib.hip after multi_wg_kernels.hip.
#include <hip/hip_runtime.h>
#include "rcd_state.h"

namespace resident {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// f(integral_constant k) for the wave-uniform k in [LO, HI): a few scalar branches, registers stay statically indexed.
// (The empty asm keeps the compiler from merging the tails of the branches into one that picks its operands through a
// pointer: an array indexed that way would live in scratch memory.)
template <int LO, int HI, typename F> __device__ __forceinline__ void at_index(int k, F &&f)
{
    if constexpr (HI - LO == 1) {
        f(std::integral_constant<int, LO>{});
        asm volatile("");
    } else {
        constexpr int MID = (LO + HI) / 2;
        if (k < MID) at_index<LO, MID>(k, f);
        else at_index<MID, HI>(k, f);
    }
}

template <int CTRL> __device__ __forceinline__ int dpp(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }

// The same for an f that changes registers: a chain of "if (k == K0) ..." that the compiler may not fold into one switch
// (k is made opaque between the tests).  Each test is a branch around an update in place; where the branches of a switch
// meet, the register allocator kept two copies of everything they change.
template <int LO, int HI, typename F> __device__ __forceinline__ void update_chain(int k, F &&f)
{
    if constexpr (LO < HI) {
        if (k == LO) f(std::integral_constant<int, LO>{});
        asm volatile("" : "+s"(k));
        update_chain<LO + 1, HI>(k, f);
    }
}
template <int LO, int HI, typename F> __device__ __forceinline__ void update_at_index(int k, F &&f)
{
    update_chain<LO, HI>(__builtin_amdgcn_readfirstlane(k), f);
}

// base[lane's 32-bit byte offset]: a scalar base and one vector register per address
template <typename V, typename T> __device__ __forceinline__ V RCD_GLOBAL *off(T RCD_GLOBAL *base, unsigned bytes)
{
    return (V RCD_GLOBAL *)((char RCD_GLOBAL *)base + (size_t)bytes);
}

// Memory read at "scalar offset + lane offset + constant": one instruction per access and one vector register
// for all of a lane's addresses.  (Through pointers every access cost a 64-bit addition and two registers.)  The matrix of
// a class that fits here is at most 16384 x 16384 floats, well below the 2 GB whose offsets fit an int.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ f32x2 buffer_load2(__amdgpu_buffer_rsrc_t b, unsigned lane_bytes, unsigned scalar_bytes)
{
    return __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(b, (int)lane_bytes, (int)scalar_bytes, 0));
}

// max over each row of 16 lanes, in every lane of the row
__device__ __forceinline__ unsigned row_max_u32(unsigned v)
{
    v = max(v, (unsigned)dpp<0xB1>((int)v));      // quad_perm 1,0,3,2
    v = max(v, (unsigned)dpp<0x4E>((int)v));      // quad_perm 2,3,0,1
    v = max(v, (unsigned)dpp<0x141>((int)v));     // row_half_mirror
    v = max(v, (unsigned)dpp<0x140>((int)v));     // row_mirror
    return v;
}

// A barrier that waits for this wave's LDS accesses and not for its loads and stores in global memory: what the waves of
// a workgroup tell each other here goes through LDS, and a wave reads back from memory only what it wrote itself.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ double max_f64(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Order-preserving key of a double (inc_key) as two words.
__device__ __forceinline__ void key_words(double x, unsigned &hi, unsigned &lo)
{
    const long long b = __double_as_longlong(x + 0.0);
    const unsigned h = (unsigned)(b >> 32), sign = (unsigned)((int)h >> 31);
    hi = h ^ (sign | 0x80000000u);
    lo = (unsigned)b ^ sign;
}

// Algorithm 1's choice of the block from the copy in the lanes (lane k & 15: block k): the least f among the blocks with
// room, lowest index on ties; -1 when every block is full.
__device__ __forceinline__ int choose_block(double f, int room)
{
    unsigned hi, lo;
    key_words(-f, hi, lo);
    if (room <= 0) hi = 0u;                      // below the key of any number
    const unsigned mhi = row_max_u32(hi);
    if (__builtin_amdgcn_readfirstlane((int)mhi) == 0) return -1;
    unsigned who = (unsigned)__ballot(hi == mhi) & 0xFFFFu;
    if (who & (who - 1u)) {
        const unsigned mlo = row_max_u32(hi == mhi ? lo : 0u);
        who = (unsigned)__ballot(hi == mhi && lo == mlo) & 0xFFFFu;
    }
    return (int)__builtin_ctz(who);
}

// A workgroup of NT threads, Q pieces of two samples per thread (at most NT * 2 Q samples), at most KM blocks.
template <int NT_, int Q_, int KM_> struct Shape {
    static constexpr int NT = NT_, Q = Q_, KM = KM_;
    static constexpr int NW = NT / 64, P = 2 * Q, WAVE = 128 * Q;
    static_assert(KM <= RCD_KMAX && (NW & (NW - 1)) == 0 && NW <= 8 && 2 * P * KM <= 192, "layout");
};

struct Slot { unsigned hi, lo; int v, pad; };

// What a wave knows about where it is.  Piece q of a lane starts at sample v0 + 128 q; pieces from nq on lie outside the
// class's pitch (a piece is wholly in or out): their gains are INC_TAKEN.  A row is read through at(), which stays inside the
// row: a class may be much smaller than the variant its launch needs for the largest.  A piece outside the pitch reads from
// the row's start instead, and what is added to INC_TAKEN for it is finite and far below its last bit.
template <typename S> struct Place {
    // one or two pieces: a wave is wholly in or out too (the pitch is a multiple of 256), and v0 alone says where it reads
    static constexpr bool WHOLE = S::Q <= 2;
    int lane, wave, nq;
    unsigned v0;
    unsigned piece[S::Q];    // bytes from a row's start to piece q of this wave (not WHOLE)
    __device__ __forceinline__ void init(int ld)
    {
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        nq = min(max((ld - wave * S::WAVE) / 128, 0), S::Q);
        v0 = (unsigned)((WHOLE && nq == 0 ? 0 : wave * S::WAVE) + lane * 2);
#pragma unroll
        for (int q = 0; q < S::Q; ++q) piece[q] = q < nq ? (unsigned)(wave * S::WAVE + 128 * q) * 4u : 0u;
    }
    // this lane's two samples of piece q in the row that starts `row` bytes into the buffer
    __device__ __forceinline__ f32x2 at(__amdgpu_buffer_rsrc_t b, unsigned row, int q) const
    {
        if constexpr (WHOLE) return buffer_load2(b, v0 * 4u, row + 512u * q);
        else return buffer_load2(b, (unsigned)lane * 8u, row + piece[q]);
    }
};

template <typename S, typename PL>
__device__ __forceinline__ void load_gains(double (&G)[S::KM][S::P], const double *g, int K, int n, int ld, const PL &pl)
{
    const double RCD_GLOBAL *src = (const double RCD_GLOBAL *)g;
#pragma unroll
    for (int k = 0; k < S::KM; ++k) {
#pragma unroll
        for (int q = 0; q < S::Q; ++q) {
            G[k][2 * q] = INC_TAKEN;
            G[k][2 * q + 1] = INC_TAKEN;
            if (k < K && q < pl.nq) {
                const int v = (int)pl.v0 + 128 * q;
                const f64x2 x = *off<const f64x2>(src + (size_t)k * ld, (unsigned)v * 8u);
                if (v < n) G[k][2 * q] = x.x;
                if (v + 1 < n) G[k][2 * q + 1] = x.y;
            }
        }
        __builtin_amdgcn_sched_barrier(0);       // a block at a time: all blocks' loads in flight would need the registers twice
    }
}

template <typename S, typename PL>
__device__ __forceinline__ void store_gains(const double (&G)[S::KM][S::P], double *g, int K, int ld, const PL &pl)
{
    double RCD_GLOBAL *dst = (double RCD_GLOBAL *)g;
#pragma unroll
    for (int k = 0; k < S::KM; ++k)
#pragma unroll
        for (int q = 0; q < S::Q; ++q)
            if (k < K && q < pl.nq) {
                const f64x2 x = {G[k][2 * q], G[k][2 * q + 1]};
                *off<f64x2>(dst + (size_t)k * ld, (pl.v0 + 128u * q) * 8u) = x;
            }
}

// The class's best candidate for block js: largest gain, lowest sample on ties (same answer in every wave).  One barrier;
// `bank` alternates between two sets of slots.  Every row of 16 lanes puts its best into a slot of its own, found by
// vector operations alone on the high word of the key (a tie there takes the long way); after the barrier every wave
// reduces the slots.  Each trip between the vector and the scalar unit costs tens of cycles in this chain, and the form
// that found the wave's best first (three wave-wide reductions) took 1.3 to 1.9 thousand cycles where this takes half.
template <typename S>
__device__ __forceinline__ void best_candidate(const double (&G)[S::KM][S::P], int js, const Place<S> &pl, Slot (*slots)[4 * S::NW],
                                               unsigned &bank, double &best, int &vstar)
{
    double m = 0.0;
    int at = 0;
    at_index<0, S::KM>(js, [&](auto kc) {
        constexpr int k = decltype(kc)::value;
        double t[S::P];
#pragma unroll
        for (int i = 0; i < S::P; ++i) t[i] = G[k][i];
#pragma unroll
        for (int w = 1; w < S::P; w *= 2)
#pragma unroll
            for (int i = 0; i + w < S::P; i += 2 * w) t[i] = max_f64(t[i], t[i + w]);
        m = t[0];
        // the lowest of the lane's samples that has it: pieces ascending, then the lane's two
        at = 0;
#pragma unroll
        for (int i = S::P - 1; i >= 1; --i) at = G[k][i] == m ? i : at;
        at = G[k][0] == m ? 0 : at;
    });
    unsigned hi, lo;
    key_words(m, hi, lo);
    const int v = pl.wave * S::WAVE + pl.lane * 2 + (at >> 1) * 128 + (at & 1);
    const unsigned top = row_max_u32(hi);
    bool win = hi == top;
    if (__popcll(__ballot(win)) != 4) {
        const unsigned low = row_max_u32(win ? lo : 0u);
        win = win && lo == low;
        const unsigned first = row_max_u32(win ? ~(unsigned)v : 0u);
        win = win && ~(unsigned)v == first;
    }
    bank ^= 1u;
    if (win) slots[bank][pl.wave * 4 + (pl.lane >> 4)] = Slot{hi, lo, v, 0};
    if constexpr (S::NW > 1) lds_barrier();
    else __builtin_amdgcn_wave_barrier();
    constexpr int N = 4 * S::NW;
    const Slot s = slots[bank][pl.lane & (N - 1)];
    unsigned g = row_max_u32(s.hi);
    if constexpr (N > 16) {
        const unsigned g0 = (unsigned)__builtin_amdgcn_readlane((int)g, 0), g1 = (unsigned)__builtin_amdgcn_readlane((int)g, 16);
        g = max(g0, g1);
    }
    constexpr unsigned long long SLOTS = (1ull << N) - 1ull;
    unsigned long long who = __ballot(s.hi == g) & SLOTS;
    if (who & (who - 1ull)) {
        const unsigned low = wave_max_u32(s.hi == g ? s.lo : 0u);
        const unsigned first = wave_max_u32(s.hi == g && s.lo == low ? ~(unsigned)s.v : 0u);
        who = __ballot(s.hi == g && s.lo == low && ~(unsigned)s.v == first) & SLOTS;
    }
    const int src = (int)__builtin_ctzll(who);
    best = inc_value(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)s.hi, src) << 32) |
                     (unsigned)__builtin_amdgcn_readlane((int)s.lo, src));
    vstar = __builtin_amdgcn_readlane(s.v, src);
}

// v* is no longer a candidate of any block: the wave that owns it (its samples start at `first`) strikes it out of its
// registers.
template <typename S>
__device__ __forceinline__ void strike(double (&G)[S::KM][S::P], int vstar, int first, int lane)
{
    const int r = vstar - first;
    if (r < 0 || r >= S::WAVE) return;           // wave-uniform
    const bool me = lane == ((r & 127) >> 1);
    update_at_index<0, S::P>((r >> 7) * 2 + (r & 1), [&](auto ic) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int k = 0; k < S::KM; ++k) {
            // the high word alone makes it a number below every live gain
            const long long b = __double_as_longlong(G[k][i]);
            const int hi = me ? (int)(__double_as_longlong(INC_TAKEN) >> 32) : (int)(b >> 32);
            G[k][i] = __longlong_as_double(((long long)hi << 32) | (b & 0xFFFFFFFFll));
        }
    });
}

// What every wave carries from pick to pick (the same in all of them).
struct Run {
    double f;                // block (lane & 15)'s f and the samples it may still take
    int room;
    int next;                // the block in turn, -1 when all are full (worked out when a pick is made, not when it is needed)
    unsigned valid;          // bit k: block k's gains are current
    int nR, t, t0, total, max_steps;
    int done, stop;          // finished; nothing more to do in this call
    int held, held_j, held_v;     // picks not yet written to the caller's arrays: lane i holds the i-th one's block and sample
};

__device__ __forceinline__ void load_run(Run &r, const RcdClass &st, int max_steps)
{
    const int k = threadIdx.x & 15;
    const bool mine = k < st.K;
    r.f = mine ? st.f[k] : 0.0;
    r.room = mine ? st.cap[k] - st.cnt[k] : 0;
    r.next = choose_block(r.f, r.room);
    r.valid = 0xFFFFu;
    r.nR = __builtin_amdgcn_readfirstlane(st.nR);
    r.t = r.t0 = __builtin_amdgcn_readfirstlane(st.t);
    r.total = __builtin_amdgcn_readfirstlane(st.total);
    r.max_steps = max_steps;
    r.done = r.stop = 0;
    r.held = r.held_j = r.held_v = 0;
}

// The block in turn if a step can be made, else -1 and the reason in done / stop.
__device__ __forceinline__ int block_in_turn(Run &r)
{
    if (r.t >= r.total || r.next < 0) { r.done = 1; return -1; }
    if (r.t - r.t0 >= r.max_steps) { r.stop = 1; return -1; }
    return r.next;
}

__device__ __forceinline__ void take(Run &r, int js, int vstar, double best, int lane)
{
    if ((lane & 15) == js) {
        r.f += best;
        r.room -= 1;
    }
    r.next = choose_block(r.f, r.room);
    if (lane == r.held) { r.held_j = js; r.held_v = vstar; }
    r.held += 1;
    r.nR -= 1;
    r.t += 1;
}

// The caller's arrays, up to 64 picks at a time, by the last wave.
template <typename S, typename PL>
__device__ __forceinline__ void write_outputs(Run &r, int32_t *assign_out, int32_t *order_out, const int32_t *out_index,
                                              const PL &pl)
{
    if (pl.wave == S::NW - 1 && pl.lane < r.held) {
        const int oi = out_index ? ((gci32)out_index)[r.held_v] : r.held_v;
        ((gi32)assign_out)[oi] = r.held_j;
        if (order_out) ((gi32)order_out)[oi] = r.t - r.held + pl.lane;
    }
    r.held = 0;
}

// The evolving part of the descriptor, by the first wave.  entries: similarity entries read; sweeps: lists left to others;
// computed: whether a step's gains count as evaluated.
__device__ __forceinline__ void store_run(const Run &r, RcdClass &st, RcdPlan *plans, long long entries, long long sweeps,
                                          bool computed, long long ticks)
{
    const int tid = threadIdx.x;
    if (tid >= 64) return;
    if (tid < st.K) {
        st.f[tid] = r.f;
        st.cnt[tid] = st.cap[tid] - r.room;
    }
    if (tid == 0) {
        st.nneed = 0;
        st.stat_sweeps += sweeps;
        st.stat_entries += entries;
        // a step looks at every candidate left: nR + steps, ..., nR + 1 of them
        const long long steps = r.t - r.t0, useful = steps * r.nR + steps * (steps + 1) / 2;
        if (computed) st.stat_computed += useful - steps;
        st.stat_steps += steps;
        st.stat_useful += useful;
        st.stat_ticks += ticks;
        st.nR = r.nR;
        st.t = r.t;
        st.done = r.done;
        if (r.done) __hip_atomic_fetch_add(&plans[0].ndone, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

} // namespace resident

// Greedy steps of one class with the graph-cut function: every marginal value of the served block drops by 2 S(v, v*).
// Two rows are on their way at any time: a row is applied when its block's turn comes again or when its registers are
// needed, two picks later.
template <typename S>
__global__ void __launch_bounds__(S::NT)
rcd_k_gc_steps_res(RcdClass *__restrict__ classes, RcdPlan *__restrict__ plans, int max_steps)
{
    using namespace resident;
    __shared__ Slot slots[2][4 * S::NW];
    RcdClass &st = classes[blockIdx.x];
    if ((st.done | plans[0].bad) != 0) return;   // (bad: the caller's S was refused.  One trip for both words.)
    const long long tick0 = wall_clock64();
    const int K = __builtin_amdgcn_readfirstlane(st.K), n = __builtin_amdgcn_readfirstlane(st.n);
    const int ld = __builtin_amdgcn_readfirstlane(st.ld);
    const __amdgpu_buffer_rsrc_t M = buffer_of(mw_uniform(st.M), n * ld * 4);
    int32_t *assign_out = mw_uniform(st.assign_out), *order_out = mw_uniform(st.order_out);
    const int32_t *out_index = mw_uniform(st.out_index);
    Place<S> pl;
    pl.init(ld);
    Run r;
    load_run(r, st, max_steps);
    double G[S::KM][S::P];
    load_gains<S>(G, inc_gains(st), K, n, ld, pl);
    unsigned bank = 0;
    f32x2 m[2][S::Q];
    int of[2] = {-1, -1};                        // block the row in flight belongs to
    auto apply = [&](auto slot) {
        constexpr int i = decltype(slot)::value;
        update_at_index<0, S::KM>(of[i], [&](auto kc) {
            constexpr int k = decltype(kc)::value;
#pragma unroll
            for (int q = 0; q < S::Q; ++q) {
                G[k][2 * q] = G[k][2 * q] - 2.0 * (double)m[i][q].x;
                G[k][2 * q + 1] = G[k][2 * q + 1] - 2.0 * (double)m[i][q].y;
            }
        });
        of[i] = -1;
    };
    auto step = [&](auto slot) {
        constexpr int i = decltype(slot)::value;
        const int js = block_in_turn(r);
        if (js < 0) return;
        if (js == of[i] || js == of[1 - i]) {
            if (of[i] >= 0) apply(std::integral_constant<int, i>{});
            if (js == of[1 - i]) apply(std::integral_constant<int, 1 - i>{});
        }
        double best;
        int vstar;
        best_candidate<S>(G, js, pl, slots, bank, best, vstar);
        if (!(best > INC_LIVE_ABOVE) || vstar >= n) { r.done = 1; return; }    // no candidate left (cannot happen while t < total <= n)
        if (of[i] >= 0) apply(std::integral_constant<int, i>{});
        const unsigned row = (unsigned)(vstar * ld) * 4u;
#pragma unroll
        for (int q = 0; q < S::Q; ++q) m[i][q] = pl.at(M, row, q);
        of[i] = js;
        strike<S>(G, vstar, pl.wave * S::WAVE, pl.lane);
        take(r, js, vstar, best, pl.lane);
    };
    while (!r.done && !r.stop) {
        asm volatile("" : "+v"(pl.v0));          // what follows from v0 is worked out where it is used, not kept for the whole loop
        step(std::integral_constant<int, 0>{});
        if (!r.done && !r.stop) step(std::integral_constant<int, 1>{});
        if (r.held >= 62 || r.done || r.stop) write_outputs<S>(r, assign_out, order_out, out_index, pl);
    }
    if (!r.done) {
        if (of[0] >= 0) apply(std::integral_constant<int, 0>{});
        if (of[1] >= 0) apply(std::integral_constant<int, 1>{});
        store_gains<S>(G, inc_gains(st), K, ld, pl);
    }
    store_run(r, st, plans, (long long)(r.t - r.t0) * n, 0, false, wall_clock64() - tick0);
}

namespace resident {

// One changed j of a pick: its old and new coverage.
struct Entry { int j; float o, n; int pad; };

__device__ __forceinline__ float max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}


// The incremental loop: BM picks at most before their updates.
template <typename S, int BM_> struct IncShape : S {
    static constexpr int BM = BM_;
    // changed j of one pick that a wave can hold in LDS; a list with a longer run in some wave is handed out
    static constexpr int STAGE = S::NT <= 256 && S::WAVE <= 128 ? S::WAVE : 64;
    // What the registers beside the gains and the sums have room for (a lane has 256 with 512 threads and 512 below): the
    // picks' own rows, kept until the lists are applied (v* is always on its own list), and rows of the lists in flight.
    static constexpr int HELD = 2 * S::P * (S::KM + 1), BUDGET = S::NT <= 256 ? 260 : 190;
    static constexpr bool OWN = HELD + BM * S::P + 4 * S::P <= BUDGET;
    static constexpr int FREE = BUDGET - HELD - (OWN ? BM * S::P : 0);
    static constexpr int ROWS = FREE >= 8 * S::P ? 8 : FREE >= 4 * S::P ? 4 : 2;
    static_assert((BM & (BM - 1)) == 0 && BM * S::NW <= 64, "a lane per wave and pick");
};

// Long update lists are handed out: the class's workgroup posts them, and helper workgroups of the same launch (and the
// class's own, when it has nothing else to do) work out the sums, 128 samples at a time.  A block has at most one list
// out.  In the class's exchange area, all read and written at device scope:
//   left[k]   slices of block k's list nobody has taken yet (taken by subtracting one; the result may run below zero)
//   ready[k]  slices finished
//   runs[k]   lengths of the list's runs (one per wave of the class's workgroup)
//   over      number of the launch in which the class's workgroup stopped: its helpers leave
// The list is in dlist / dold / dnew, the sums go to HELP_SUMS.  Nobody waits for a workgroup that may not be running: what
// no helper has taken, the class's workgroup takes itself, and it waits only for slices in work.
// (HP_LEFT, which helpers poll and the class's workgroup sets, in another 128-byte line than HP_READY, which they add to: in one line
// ten classes of 5000 take 1 % longer.  HP_OVER, which they poll too, lies beside HP_READY.)
enum { HP_LEFT = MW_SLOT + 16, HP_READY = HP_LEFT + RCD_KMAX, HP_OVER = HP_READY + RCD_KMAX, HP_RUNS = HP_OVER + 16,
       HP_END = HP_RUNS + 8 * RCD_KMAX };
static_assert(HP_END <= MW_PEND && RCD_MW_INTS % 32 == 0, "exchange area too small");
static_assert((HP_LEFT + RCD_KMAX - 1) / 32 < HP_READY / 32, "two lines");

struct Lists {
    gi32 box;                // the class's exchange area
    gi32 j;
    gf32 o, n;               // K x ld each: changed j, old and new coverage, run w from w * WAVE on
    double RCD_GLOBAL *sums; // K x ld
    int ld, slices;
    __device__ __forceinline__ void init(const RcdClass &st)
    {
        ld = __builtin_amdgcn_readfirstlane(st.ld);
        slices = ld / 128;
        box = (gi32)mw_uniform(st.mwbuf);
        j = (gi32)mw_uniform(inc_dlist(st));
        o = (gf32)mw_uniform(inc_dold(st));
        n = (gf32)mw_uniform(inc_dnew(st));
        sums = (double RCD_GLOBAL *)(mw_uniform(inc_gains(st)) + 2 * (size_t)st.K * ld);
    }
};

// One slice of block k's list, if one is left: true when it was done.  Called by one wave.
template <typename S, int U>
__device__ __forceinline__ bool help_once(const Lists &li, const __amdgpu_buffer_rsrc_t M, int k, int lane)
{
    int mine = 0;
    __builtin_amdgcn_wave_barrier();
    if (lane == 0) mine = __hip_atomic_fetch_add(li.box + HP_LEFT + k, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    mine = __builtin_amdgcn_readfirstlane(mine);
    if (mine <= 0) return false;
    const unsigned part = (unsigned)(mine - 1) * 512u;
    const int len = lane < S::NW ? dev_load(li.box + HP_RUNS + 8 * k + lane) : 0;
    int nd = 0;
#pragma unroll
    for (int w = 0; w < S::NW; ++w) nd += __builtin_amdgcn_readlane(len, w);
    double a0 = 0.0, a1 = 0.0;
    for (int first = 0; first < nd; first += 64) {
        int at = k * li.ld, start = first + lane;
        bool found = false;
#pragma unroll
        for (int w = 0; w < S::NW; ++w) {
            const int c = __builtin_amdgcn_readlane(len, w);
            if (!found && start < c) { at += w * S::WAVE + start; found = true; }
            start -= c;
        }
        int ej = 0;
        float eo = 0.f, en = 0.f;
        if (found) {
            ej = dev_load(li.j + at);
            eo = dev_load(li.o + at);
            en = dev_load(li.n + at);
        }
        const unsigned row_of = (unsigned)(ej * li.ld) * 4u + part;
        const int here = min(64, nd - first);
        for (int e0 = 0; e0 < here; e0 += U) {
            f32x2 m[U];
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (e0 + i < here) m[i] = buffer_load2(M, (unsigned)lane * 8u, (unsigned)__builtin_amdgcn_readlane((int)row_of, e0 + i));
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (e0 + i < here) {
                    const float cn = inc_lane_value(en, e0 + i), co = inc_lane_value(eo, e0 + i);
                    a0 += inc_term(m[i].x, cn, co);
                    a1 += inc_term(m[i].y, cn, co);
                }
        }
    }
    unsigned long long RCD_GLOBAL *out = (unsigned long long RCD_GLOBAL *)(li.sums + (size_t)k * li.ld + (mine - 1) * 128 + lane * 2);
    __hip_atomic_store(out, (unsigned long long)__double_as_longlong(a0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(out + 1, (unsigned long long)__double_as_longlong(a1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_for_my_stores();
    if (lane == 0) __hip_atomic_fetch_add(li.box + HP_READY + k, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // The wave stays together: without this the compiler ran "lane 0 again" of a caller's loop straight into the next
    // attempt's "lane 0", ahead of the other lanes, which then saw no slice to take.
    __builtin_amdgcn_wave_barrier();
    return true;
}

// A helper wave: takes slices of its class's lists until the class's workgroup has stopped (or nothing has come for
// spin_ticks: the class then serves itself).
template <typename S>
__device__ __forceinline__ void help(const RcdClass &st, int launch, long long spin_ticks)
{
    Lists li;
    li.init(st);
    const int lane = threadIdx.x & 63;
    const int K = __builtin_amdgcn_readfirstlane(st.K);
    const __amdgpu_buffer_rsrc_t M = buffer_of(mw_uniform(st.M), __builtin_amdgcn_readfirstlane(st.n) * li.ld * 4);
    long long deadline = wall_clock64() + spin_ticks;
    for (;;) {
        const int word = lane < K ? dev_load(li.box + HP_LEFT + lane) : lane == 63 ? dev_load(li.box + HP_OVER) : 0;
        if (__builtin_amdgcn_readlane(word, 63) == launch) return;
        const unsigned some = (unsigned)__ballot(lane < K && word > 0);
        if (some) {
            if (help_once<S, 32>(li, M, (int)__builtin_ctz(some), lane)) deadline = wall_clock64() + spin_ticks;
        } else {
            if (wall_clock64() > deadline) return;
            __builtin_amdgcn_s_sleep(8);
        }
    }
}

// Block k's list is out and its turn has come: this workgroup's waves take what slices are left, wait for those in work
// (bounded) and add the sums to the block's gains.
template <typename S>
__device__ __forceinline__ bool collect(double (&G)[S::KM][S::P], int k, const Lists &li, const __amdgpu_buffer_rsrc_t M,
                                        const Place<S> &pl, int *abort_flag, int *s_fail, long long spin_ticks)
{
    while (help_once<S, 4>(li, M, k, pl.lane)) {}
    const long long deadline = wall_clock64() + spin_ticks;
    int ok = 1;
    while (dev_load(li.box + HP_READY + k) < li.slices) {
        if (__hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2 || wall_clock64() > deadline) {
            __hip_atomic_store(abort_flag, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = 0;
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    if constexpr (S::NW > 1) {
        if (!ok) *s_fail = 1;
        lds_barrier();
        ok = *s_fail == 0;
    }
    if (!ok) return false;
    const unsigned long long RCD_GLOBAL *src = (const unsigned long long RCD_GLOBAL *)(li.sums + (size_t)k * li.ld);
    double sum[S::P];
#pragma unroll
    for (int q = 0; q < S::Q; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            sum[2 * q + c] = 0.0;
            if (q < pl.nq)
                sum[2 * q + c] = __longlong_as_double((long long)__hip_atomic_load(src + pl.v0 + 128 * q + c, __ATOMIC_RELAXED,
                                                                                   __HIP_MEMORY_SCOPE_AGENT));
        }
    update_at_index<0, S::KM>(k, [&](auto kc) {
        constexpr int kk = decltype(kc)::value;
#pragma unroll
        for (int i = 0; i < S::P; ++i) G[kk][i] += sum[i];
    });
    return true;
}

} // namespace resident

// Greedy steps of one class on the incremental route.  A batch: up to BM picks, each pick's row v* asked for when it is
// made; then the rows against their blocks' coverage, and per pick the ordered list of changed j; one barrier; then the
// rows of the lists that are short enough, all picks' lists end to end (ROWS rows in flight).  A longer list is handed out
// to the workgroups from ncls on (helper_of says which class each of them serves; without it they take the classes one
// after the other); its block waits for the sums when its turn comes.
template <typename S>
__global__ void __launch_bounds__(S::NT)
rcd_k_inc_steps_res(RcdClass *__restrict__ classes, RcdPlan *__restrict__ plans, const RcdWg *__restrict__ helper_of,
                    int ncls, int max_steps, int small_bytes, int launch, long long spin_ticks)
{
    using namespace resident;
    constexpr int NW = S::NW, Q = S::Q, P = S::P, STAGE = S::STAGE;
    __shared__ Slot slots[2][4 * NW];
    __shared__ __attribute__((aligned(16))) Entry stage[S::BM * NW][STAGE];
    __shared__ int scount[S::BM * NW];
    __shared__ int s_fail;
    const int wg = (int)blockIdx.x;
    const int cls = wg < ncls ? wg : helper_of ? helper_of[wg - ncls].cls : wg % ncls;
    RcdClass &st = classes[__builtin_amdgcn_readfirstlane(cls)];
    // (bad: the caller's S was refused, and one launch would run the whole class before the host hears of it; or a wait of
    // the launch before ran out, whose state was not stored.  One trip to memory for both words.)
    if ((st.done | plans[0].bad) != 0) return;
    if (wg >= ncls) {
        help<S>(st, launch, spin_ticks);
        return;
    }
    const long long tick0 = wall_clock64();
    const int K = __builtin_amdgcn_readfirstlane(st.K), n = __builtin_amdgcn_readfirstlane(st.n);
    const int ld = __builtin_amdgcn_readfirstlane(st.ld);
    const __amdgpu_buffer_rsrc_t M = buffer_of(mw_uniform(st.M), n * ld * 4);
    const __amdgpu_buffer_rsrc_t cover = buffer_of(mw_uniform(st.cur), K * ld * 4);
    const gf32 cur_all = (gf32)mw_uniform(st.cur);
    Lists li;
    li.init(st);
    int32_t *assign_out = mw_uniform(st.assign_out), *order_out = mw_uniform(st.order_out);
    const int32_t *out_index = mw_uniform(st.out_index);
    // lists up to this many rows are applied right here
    const int small = max(4, min(NW * STAGE, small_bytes / (ld * 4)));
    Place<S> pl;
    pl.init(ld);
    const int lane = pl.lane;
    const unsigned long long below = (1ull << lane) - 1ull;
    Run r;
    load_run(r, st, max_steps);
    if (threadIdx.x == 0) s_fail = 0;          // (first read behind a barrier of a pick or of collect())
    double G[S::KM][P];
    load_gains<S>(G, inc_gains(st), K, n, ld, pl);
    unsigned bank = 0;
    bool alive = true;
    long long entries = 0, sweeps = 0;           // entries: this lane's share of the list lengths
    while (!r.done && !r.stop) {
        if (r.next >= 0 && !((r.valid >> r.next) & 1u) && r.t < r.total) {
            if (!collect<S>(G, r.next, li, M, pl, &plans[0].bad, &s_fail, spin_ticks)) { alive = false; break; }
            r.valid |= 1u << r.next;
        }
        asm volatile("" : "+v"(pl.v0));          // what follows from v0 is worked out where it is used, not kept for the whole loop
        int B = 0;
        int pj[S::BM], pv[S::BM];                // the picks' blocks and samples
        f32x2 mp[S::BM][Q];                      // their rows
        {
            // ---- picks
            unsigned busy = 0;
            bool more = true;
#pragma unroll
            for (int u = 0; u < S::BM; ++u) {
                pj[u] = 0;
                pv[u] = -1;
                if (more) {
                    const int js = block_in_turn(r);
                    more = js >= 0 && !((busy >> js) & 1u) && ((r.valid >> js) & 1u);
                    if (more) {
                        double best;
                        int vstar;
                        best_candidate<S>(G, js, pl, slots, bank, best, vstar);
                        if (!(best > INC_LIVE_ABOVE) || vstar >= n) {    // no candidate left (cannot happen while t < total <= n)
                            r.done = 1;
                            more = false;
                        } else {
                            const unsigned row = (unsigned)(vstar * ld) * 4u;
#pragma unroll
                            for (int q = 0; q < Q; ++q) mp[u][q] = pl.at(M, row, q);
                            strike<S>(G, vstar, pl.wave * S::WAVE, pl.lane);
                            take(r, js, vstar, best, lane);
                            busy |= 1u << js;
                            pj[u] = js;
                            pv[u] = vstar;
                            B = u + 1;
                        }
                    }
                }
            }
            if (B == 0) break;

            // ---- coverage: the j of this wave's samples with S(j, v*) > cur_k(j), ascending, into LDS
            f32x2 c[S::BM][Q];
#pragma unroll
            for (int u = 0; u < S::BM; ++u)
                if (u < B) {
                    const unsigned row = (unsigned)(pj[u] * ld) * 4u;
#pragma unroll
                    for (int q = 0; q < Q; ++q) c[u][q] = pl.at(cover, row, q);
                }
#pragma unroll
            for (int u = 0; u < S::BM; ++u)
                if (u < B) {
                    const size_t row_k = (size_t)pj[u] * ld, at = row_k + pl.wave * S::WAVE;
                    Entry *held = stage[u * NW + pl.wave];
                    int cnt = 0;
#pragma unroll
                    for (int q = 0; q < Q; ++q)
                        if (q < pl.nq) {
                            const bool ch0 = mp[u][q].x > c[u][q].x, ch1 = mp[u][q].y > c[u][q].y;
                            const unsigned long long b0 = __ballot(ch0), b1 = __ballot(ch1);
                            if ((b0 | b1) != 0ull) {
                                const int v = (int)pl.v0 + 128 * q;
                                unsigned pos = cnt + __popcll(b0 & below) + __popcll(b1 & below);
                                auto keep = [&](int j, float old_c, float new_c) {
                                    if (pos < STAGE) {
                                        held[pos] = Entry{j, old_c, new_c, 0};
                                    } else {         // a run too long to be held: this list is handed out
                                        dev_store(li.j + at + pos, j);
                                        dev_store(li.o + at + pos, old_c);
                                        dev_store(li.n + at + pos, new_c);
                                        *off<float>(cur_all + row_k, (unsigned)j * 4u) = new_c;
                                    }
                                    ++pos;
                                };
                                if (ch0) keep(v, c[u][q].x, mp[u][q].x);
                                if (ch1) keep(v + 1, c[u][q].y, mp[u][q].y);
                                cnt += __popcll(b0) + __popcll(b1);
                            }
                        }
                    if (lane == 0) scount[u * NW + pl.wave] = cnt;
                }
        }
        if constexpr (NW > 1) lds_barrier();
        else __builtin_amdgcn_wave_barrier();

        // ---- the lists: lane u NW + w holds the length of wave w's run for pick u
        const int found = lane < B * NW ? scount[lane & (S::BM * NW - 1)] : 0;
        entries += found;
        int nd = found, longest = found;          // over the pick's NW runs
        if constexpr (NW > 1) { nd += dpp<0xB1>(nd); longest = max(longest, dpp<0xB1>(longest)); }
        if constexpr (NW > 2) { nd += dpp<0x4E>(nd); longest = max(longest, dpp<0x4E>(longest)); }
        if constexpr (NW > 4) { nd += dpp<0x141>(nd); longest = max(longest, dpp<0x141>(longest)); }
        const bool pending = nd > small || longest > STAGE;
        const unsigned long long left_over = __ballot(pending);
        const int cnt = pending ? 0 : found;
        int incl = cnt;                           // inclusive prefix over the lanes
        incl += dpp<0x111>(incl);
        incl += dpp<0x112>(incl);
        incl += dpp<0x114>(incl);
        incl += dpp<0x118>(incl);
        {
            const int r0 = __builtin_amdgcn_readlane(incl, 15), r1 = __builtin_amdgcn_readlane(incl, 31);
            const int r2 = __builtin_amdgcn_readlane(incl, 47);
            incl += (lane >= 16 ? r0 : 0) + (lane >= 32 ? r1 : 0) + (lane >= 48 ? r2 : 0);
        }
        const int excl = incl - cnt;
        const int total = __builtin_amdgcn_readlane(incl, 63);

        // ---- gains: the lists' terms, all picks' lists end to end, added up per pick in list order, then onto the block's gains
        double acc[P];
        int of = -1;                              // pick the sums are for
        auto flush = [&]() {
            int k = pj[0];
#pragma unroll
            for (int u = 1; u < S::BM; ++u) k = of == u ? pj[u] : k;
            if (of >= 0)
                update_at_index<0, S::KM>(k, [&](auto kc) {
                    constexpr int kk = decltype(kc)::value;
#pragma unroll
                    for (int i = 0; i < P; ++i) G[kk][i] += acc[i];
                });
        };
        for (int first = 0; first < total; first += 64) {
            // lane i fetches entry first + i: the run it falls into, and its place in it
            int run = 0, rel = 0;
            if (total < 64) {
                // every run tells the lane of its first entry its number; a lane looks for the last such lane up to itself
                const int got = __builtin_amdgcn_ds_permute((cnt > 0 ? excl : 63) * 4, cnt > 0 ? lane + 1 : 0);
                const unsigned long long starts = __ballot(got != 0);
                const int s = 63 - __builtin_clzll((starts & ((2ull << lane) - 1ull)) | 1ull);
                const int mine = __builtin_amdgcn_ds_bpermute(s * 4, got) - 1;
                if (lane < total) { run = mine; rel = lane - s; }
            } else {
                for (unsigned long long left = __ballot(cnt > 0); left; left &= left - 1ull) {
                    const int s = (int)__builtin_ctzll(left);
                    const int x = first + lane - __builtin_amdgcn_readlane(excl, s);
                    if (x >= 0 && x < __builtin_amdgcn_readlane(cnt, s)) { run = s; rel = x; }
                }
            }
            const Entry en = stage[run][rel];
            const int pick = run / NW;
            const unsigned row_of = (unsigned)(en.j * ld) * 4u;
            const int here = min(64, total - first);
            // the first entry of each pick, and the entries that are a pick's own row
            const int before = __builtin_amdgcn_update_dpp(-1, pick, 0x138, 0xF, 0xF, false);      // the lane below's (wave shift)
            const unsigned long long turns = __ballot(pick != before);
            unsigned long long own = 0ull;
            if constexpr (S::OWN) {
                int v = pv[0];
#pragma unroll
                for (int u = 1; u < S::BM; ++u) v = pick == u ? pv[u] : v;
                own = __ballot(en.j == v);
            }
            // U rows at a time, all asked for before the first is used
            constexpr int U = S::ROWS;
            for (int e0 = 0; e0 < here; e0 += U) {
                f32x2 m[U][Q];
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (e0 + i < here) {
                        if (S::OWN && ((own >> (e0 + i)) & 1ull)) {
                            const int u = __builtin_amdgcn_readlane(pick, e0 + i);
                            update_at_index<0, S::BM>(u, [&](auto uc) {
#pragma unroll
                                for (int q = 0; q < Q; ++q) m[i][q] = mp[decltype(uc)::value][q];
                            });
                        } else {
                            const unsigned row = (unsigned)__builtin_amdgcn_readlane((int)row_of, e0 + i);
#pragma unroll
                            for (int q = 0; q < Q; ++q) m[i][q] = pl.at(M, row, q);
                        }
                    }
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (e0 + i < here) {
                        if ((turns >> (e0 + i)) & 1ull) {
                            const int u = __builtin_amdgcn_readlane(pick, e0 + i);
                            if (u != of) {
                                flush();
                                of = u;
#pragma unroll
                                for (int x = 0; x < P; ++x) acc[x] = 0.0;
                            }
                        }
                        const float cn = inc_lane_value(en.n, e0 + i), co = inc_lane_value(en.o, e0 + i);
                        bool any = true;
                        if constexpr (P >= 6) {
                            // a sample no nearer to j than j's old coverage has no term; late in a run that is nearly all of them
                            float far = max3(m[i][0].x, m[i][0].y, co);
#pragma unroll
                            for (int q = 1; q < Q; ++q) far = max3(m[i][q].x, m[i][q].y, far);
                            any = __ballot(far > co) != 0ull;
                        }
                        if (any) {
#pragma unroll
                            for (int q = 0; q < Q; ++q) {
                                acc[2 * q] += inc_term(m[i][q].x, cn, co);
                                acc[2 * q + 1] += inc_term(m[i][q].y, cn, co);
                            }
                        }
                    }
            }
        }
        flush();

        // ---- the new coverage of this wave's samples, and the lists that are handed out, out of LDS (kept
        //      until now so that no load above waits behind a store)
#pragma unroll
        for (int u = 0; u < S::BM; ++u)
            if (u < B) {
                const size_t row_k = (size_t)pj[u] * ld, at = row_k + pl.wave * S::WAVE;
                const int mine = min(__builtin_amdgcn_readlane(found, u * NW + pl.wave), STAGE);
                const bool listed = (left_over >> (u * NW)) & 1ull;
                for (int e = lane; e < mine; e += 64) {
                    const Entry en = stage[u * NW + pl.wave][e];
                    *off<float>(cur_all + row_k, (unsigned)en.j * 4u) = en.n;
                    if (listed) {
                        dev_store(li.j + at + e, en.j);
                        dev_store(li.o + at + e, en.o);
                        dev_store(li.n + at + e, en.n);
                    }
                }
            }
        if (left_over != 0ull) {
            // post them: the lists have left this compute unit, then the run lengths, then the slices are up for taking
            wait_for_my_stores();
            if constexpr (NW > 1) lds_barrier();
#pragma unroll
            for (int u = 0; u < S::BM; ++u)
                if ((left_over >> (u * NW)) & 1ull) {
                    r.valid &= ~(1u << pj[u]);
                    sweeps += 1;
                    if (pl.wave == 0) {
                        if (lane / NW == u) dev_store(li.box + HP_RUNS + 8 * pj[u] + (lane & (NW - 1)), found);
                        if (lane == 0) dev_store(li.box + HP_READY + pj[u], 0);
                    }
                }
            if (pl.wave == 0) {
                wait_for_my_stores();
#pragma unroll
                for (int u = 0; u < S::BM; ++u)
                    if (((left_over >> (u * NW)) & 1ull) && lane == 0) dev_store(li.box + HP_LEFT + pj[u], li.slices);
            }
            // (collect() starts with an attempt to take a slice: it must not come before the post of another wave)
            if constexpr (NW > 1) lds_barrier();
        }
        if (r.held > 64 - S::BM) write_outputs<S>(r, assign_out, order_out, out_index, pl);
    }
    // the state goes to memory whole: no list stays out
    for (int k = 0; alive && !r.done && k < K; ++k)
        if (!((r.valid >> k) & 1u)) {
            alive = collect<S>(G, k, li, M, pl, &plans[0].bad, &s_fail, spin_ticks);
            r.valid |= 1u << k;
        }
    if (threadIdx.x == 0) dev_store(li.box + HP_OVER, launch);
    if (!alive) return;          // a bounded wait ran out: plans[0].bad says so, nothing is written back
    write_outputs<S>(r, assign_out, order_out, out_index, pl);
    if (!r.done) store_gains<S>(G, inc_gains(st), K, ld, pl);
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) entries += __shfl_xor(entries, x);
    store_run(r, st, plans, entries * n, sweeps, true, wall_clock64() - tick0);
}

namespace resident {

// The variants for a group whose largest class has pitch ld (samples rounded up to 256) and K blocks: the smallest that
// holds the class.  Graph cut: null beyond 2 P KM = 192 registers of gains per lane (of 256 with 512 threads); six pieces and
// eight blocks, the most, spill a few in the loop (8 of its accesses go to scratch memory).
struct Choice {
    void (*gc)(RcdClass *, RcdPlan *, int);
    void (*inc)(RcdClass *, RcdPlan *, const RcdWg *, int, int, int, int, long long);
    int threads;
};

template <int NT, int Q, int KM> Choice gc_choice() { return Choice{rcd_k_gc_steps_res<Shape<NT, Q, KM>>, nullptr, NT}; }
template <int NT, int Q, int KM, int BM> Choice inc_choice()
{
    return Choice{nullptr, rcd_k_inc_steps_res<IncShape<Shape<NT, Q, KM>, BM>>, NT};
}

inline Choice choose_gc(int ld, int K)
{
    if (ld <= 256) return gc_choice<64, 2, 16>();
    if (ld <= 512) return gc_choice<128, 2, 16>();
    if (ld <= 1024) return gc_choice<256, 2, 16>();
    if (ld <= 2048) return gc_choice<512, 2, 16>();
    if (ld <= 3072) return K <= 8 ? gc_choice<512, 3, 8>() : gc_choice<512, 3, 16>();
    if (ld <= 4096 && K > 8 && K <= 12) return gc_choice<512, 4, 12>();
    if (ld <= 5120 && K <= 8) return K <= 4 ? gc_choice<512, 5, 4>() : gc_choice<512, 5, 8>();
    if (ld <= 6144 && K > 4 && K <= 8) return gc_choice<512, 6, 8>();
    if (ld <= 8192 && K <= 4) return gc_choice<512, 8, 4>();
    if (ld <= 16384 && K <= 2) return gc_choice<512, 16, 2>();
    return Choice{nullptr, nullptr, 0};
}

// Against rcd_k_inc_steps (whole calls, start of its launches to their end, before -> after in ms): ten classes of 5000 and
// four blocks 44.9 -> 25.5, eight blocks 49.2 -> 40.5, one such class 38.8 -> 35.0; four classes of 3000, eight blocks
// 22.2 -> 13.7; 8000 samples, four blocks 73.7 -> 67.6; thirty of 2000, sixteen blocks 20.7 -> 12.1; a hundred of 500
// 8.3 -> 3.4.  Not taken, because the gains leave too few registers for the rest and the loop spills too much: 3072 samples
// and sixteen blocks (22.4 -> 25.9), 6144 and eight (51.8 -> 62.7).  (5120 and eight, 8192 and four spill as well, 24 and 31
// registers.)
inline Choice choose_inc(int ld, int K)
{
    if (ld <= 256) return inc_choice<128, 1, 16, 4>();
    if (ld <= 512) return inc_choice<256, 1, 16, 4>();
    if (ld <= 1024) return inc_choice<512, 1, 16, 2>();
    if (ld <= 2048) return inc_choice<512, 2, 16, 2>();
    if (ld <= 3072 && K <= 8) return inc_choice<512, 3, 8, 2>();
    if (ld <= 5120 && K <= 8) return K <= 4 ? inc_choice<512, 5, 4, 2>() : inc_choice<512, 5, 8, 1>();
    if (ld <= 8192 && K <= 4) return inc_choice<512, 8, 4, 1>();
    return Choice{nullptr, nullptr, 0};
}

} // namespace resident
