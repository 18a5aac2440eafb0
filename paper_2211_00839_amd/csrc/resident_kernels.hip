// Step loop of the graph-cut function that keeps a class's gains in registers (gfx950), one workgroup per class, for
// classes of up to a few thousand samples.
//
// What bounds the loop is latency: a step is a chain of a scan, a reduction and a trip to memory for row v* of S.  The loop
// of incremental_kernels.hip walks that chain once per step with the gains in L2.  Here
//   - the gains of all blocks sit in the registers of the workgroup (n x K doubles: 160 KB for 5000 samples and four
//     blocks, of the 512 KB a compute unit has), so the scan is arithmetic;
//   - the block state (f, room left) sits in the lanes of every wave, so choosing the block is one wave reduction;
//   - picks run ahead of updates.  Taking v* into block k changes the gains of block k only (and strikes v* out
//     everywhere), so the next block's argmax can be taken while row v* is still on its way, unless that block is k again.
// The order of the steps, every sum and every tie are those of the other loop: the results are the same bits.
// Measured, one class, us per step before -> after: 250 samples and 2 blocks 2.25 -> 0.90, 1000 / 8 2.28 -> 0.98,
// 3000 / 8 2.54 -> 0.99, 5000 / 4 3.14 -> 1.14; ten classes of 5000 with 4 blocks, whole call 18.7 -> 7.2 ms.  What is left
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
// class's pitch (a piece is wholly in or out): their gains are INC_TAKEN, and what is read for them is not used.
template <typename S> struct Place {
    int lane, wave, nq;
    unsigned v0;
    __device__ __forceinline__ void init(int ld)
    {
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        nq = min(max((ld - wave * S::WAVE) / 128, 0), S::Q);
        v0 = (unsigned)(wave * S::WAVE + lane * 2);
    }
};

template <typename S>
__device__ __forceinline__ void load_gains(double (&G)[S::KM][S::P], const double *g, int K, int n, int ld, const Place<S> &pl)
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

template <typename S>
__device__ __forceinline__ void store_gains(const double (&G)[S::KM][S::P], double *g, int K, int ld, const Place<S> &pl)
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

// v* is no longer a candidate of any block: the wave that owns it strikes it out of its registers.
template <typename S>
__device__ __forceinline__ void strike(double (&G)[S::KM][S::P], int vstar, const Place<S> &pl)
{
    const int r = vstar - pl.wave * S::WAVE;
    if (r < 0 || r >= S::WAVE) return;           // wave-uniform
    const bool me = pl.lane == ((r & 127) >> 1);
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
template <typename S>
__device__ __forceinline__ void write_outputs(Run &r, int32_t *assign_out, int32_t *order_out, const int32_t *out_index,
                                              const Place<S> &pl)
{
    if (pl.wave == S::NW - 1 && pl.lane < r.held) {
        const int oi = out_index ? ((gci32)out_index)[r.held_v] : r.held_v;
        ((gi32)assign_out)[oi] = r.held_j;
        if (order_out) ((gi32)order_out)[oi] = r.t - r.held + pl.lane;
    }
    r.held = 0;
}

// The evolving part of the descriptor, by the first wave.  entries: similarity entries read.
__device__ __forceinline__ void store_run(const Run &r, RcdClass &st, RcdPlan *plans, long long entries, long long ticks)
{
    const int tid = threadIdx.x;
    if (tid >= 64) return;
    if (tid < st.K) {
        st.f[tid] = r.f;
        st.cnt[tid] = st.cap[tid] - r.room;
    }
    if (tid == 0) {
        st.nneed = 0;
        st.stat_entries += entries;
        // a step looks at every candidate left: nR + steps, ..., nR + 1 of them
        const long long steps = r.t - r.t0, useful = steps * r.nR + steps * (steps + 1) / 2;
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
    if (st.done) return;
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
        for (int q = 0; q < S::Q; ++q) m[i][q] = buffer_load2(M, pl.v0 * 4u, row + 512u * q);
        of[i] = js;
        strike<S>(G, vstar, pl);
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
    store_run(r, st, plans, (long long)(r.t - r.t0) * n, wall_clock64() - tick0);
}

namespace resident {

// The variant for a group whose largest class has pitch ld (samples rounded up to 256) and K blocks: the smallest that
// holds the class; null beyond 2 P KM = 192 registers of gains per lane (of 256 with 512 threads), the most that compiles
// without spilling in the loop.
struct Choice {
    void (*gc)(RcdClass *, RcdPlan *, int);
    int threads;
};

template <int NT, int Q, int KM> Choice choice_of() { return Choice{rcd_k_gc_steps_res<Shape<NT, Q, KM>>, NT}; }

inline Choice choose(int ld, int K)
{
    if (ld <= 256) return choice_of<64, 2, 16>();
    if (ld <= 512) return choice_of<128, 2, 16>();
    if (ld <= 1024) return choice_of<256, 2, 16>();
    if (ld <= 2048) return choice_of<512, 2, 16>();
    if (ld <= 3072) return K <= 8 ? choice_of<512, 3, 8>() : choice_of<512, 3, 16>();
    if (ld <= 4096 && K > 8 && K <= 12) return choice_of<512, 4, 12>();
    if (ld <= 5120 && K <= 8) return K <= 4 ? choice_of<512, 5, 4>() : choice_of<512, 5, 8>();
    if (ld <= 6144 && K > 4 && K <= 8) return choice_of<512, 6, 8>();
    if (ld <= 8192 && K <= 4) return choice_of<512, 8, 4>();
    if (ld <= 16384 && K <= 2) return choice_of<512, 16, 2>();
    return Choice{nullptr, 0};
}

} // namespace resident
