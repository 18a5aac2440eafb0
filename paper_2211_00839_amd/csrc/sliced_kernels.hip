// Step loop of the incremental-gain route for classes that are too large for one workgroup's registers (gfx950): W
// workgroups share a class, each with its slice of the samples, whose gains it holds in registers, and up to eight picks
// share the trips between the workgroups.
//
// What bounds a step of a shared class is waiting: the workgroups tell each other their best candidates, fetch row v* of
// S, tell each other which coverage values rose, fetch the rows of that list.  rcd_k_inc_steps_mw walks this chain once per
// step, with the gains in L2.  Here
//   - the slice's gains sit in registers (512 threads hold up to 2048 samples x 8 blocks or 1024 x 16; up to 64 workgroups to a
//     class of up to 65 536 samples, larger ones are the older loop's), so the scan is arithmetic (as in resident_kernels.hip, whose
//     helpers this loop uses);
//   - a trip makes up to eight picks, all on the gains as they are at its start.  f never falls, so the u-th pick goes to one of the
//     u least blocks: every workgroup posts its best candidates of the eight least blocks (two of each, four or eight where fewer
//     blocks are left), and Algorithm 1 runs on the class's best of them, alike in every workgroup, until a list ends;
//   - a block may be picked again in the same trip.  A gain only falls, so the best of the old gains is the best of the
//     new ones if its own has not fallen, and it has not if no coverage that the block's earlier picks of the trip raise is below
//     its similarity.  That is looked up once the lists are known; the first guess that does not hold and the picks behind it
//     are dropped, and nothing has been written for them.  A class remembers how many held and guesses as far as that pays
//     (sliced_guess.h), and looks at twice as many blocks as the last trip served: where every sample has a near copy, most fail.
//     Always as far as there are candidates -> this: such pairs, one class of 6000, one block 67 -> 40 ms, 20 000, one 222 -> 138;
//     mixtures 26.5 -> 23.3, 78.6 -> 74.3.
// Picks, sums and ties are those of the other loops, in their order: the results are the same bits.
// On mixtures a trip makes 7.8 steps.  With two picks to a trip -> now, whole calls in ms on mixtures of 64 features (inc_update_narrow's
// part in it: 5 to 10 %): 50 000 samples and eight blocks 421 -> 246, 20 000 and eight 139 -> 83, one 141 -> 74, 12 000 and four 71 -> 47,
// 6000 and three 32 -> 23.  A trip at 50 000 takes 24.6 us in a copy that keeps clocks: candidates 1.9, first exchange 5.0, the
// picks 3.4, their rows and lists 2.0, second exchange 4.1, the lists' rows 6.1, the rest 1.2; an instruction of a wave
// takes some seven cycles here, so the picks' and the exchanges' arithmetic counts as much as the trips through memory.
// The tags, banks and bounded waits of the exchanges are those of multi_wg_kernels.hip; a post has sixteen pieces.
// Included by rcd_lib.hip after resident_kernels.hip.
#include <hip/hip_runtime.h>
#include "rcd_state.h"
#include "sliced_guess.h"
#include "sliced_post.h"

namespace sliced {

using resident::Entry;
using resident::Run;
using resident::Shape;
using resident::Slot;
using resident::f32x2;
using resident::lds_barrier;
using resident::off;

// 512 threads, Q pieces of two samples each, at most KM blocks, twice ROWS rows of the lists in flight.  (Q = 2 with eight rows and
// two sets of them would spill more of the picks' rows, which makes a wait of each spill: 32 registers are spilled with eight
// blocks and ROWS = 4, four with four blocks, and two of <1, 16, 8>.)
// LEARN: guesses are made as far as they hold.  With more than eight blocks a trip's picks go to eight of them and guesses are rare:
// keeping count took 0.1 to 0.9 % of a call and gave nothing (6000, sixteen blocks 28.6 / 28.8 ms, every sample with a near copy, ten of 5000
// 40.7 / 40.8).
template <int Q, int KM, int ROWS_> struct SliceShape : Shape<512, Q, KM> {
    static constexpr int ROWS = ROWS_;
    static constexpr bool LEARN = KM <= BM;
};

// Where a wave is: it owns the class's samples [first, first + 128 Q), pieces from nq on lie outside the slice.  A row is
// read through at(): a piece outside reads the wave's own place in the slice's first wave instead, so no address leaves the row.
template <typename S> struct SlicePlace {
    int lane, wave, nq, first;
    unsigned v0;             // this lane's first sample
    unsigned piece[S::Q];    // bytes from a row's start to piece q of this wave
    __device__ __forceinline__ void init(int s0, int s1)
    {
        lane = threadIdx.x & 63;
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        first = s0 + wave * S::WAVE;
        nq = min(max((s1 - first) / 128, 0), S::Q);
        v0 = (unsigned)(first + lane * 2);
#pragma unroll
        for (int q = 0; q < S::Q; ++q) piece[q] = (unsigned)(q < nq ? first + 128 * q : s0) * 4u;
    }
    __device__ __forceinline__ f32x2 at(gcf32 row, int q) const
    {
        return *off<const f32x2>((const char RCD_GLOBAL *)row + piece[q], (unsigned)lane * 8u);
    }
};

constexpr int POST_INTS = 4 * POST;
static_assert(2 * POST_INTS == RCD_SLICE_INTS && ENTRIES >= INC_SMALL && RCD_SLICES_MAX <= 64, "exchange area, a lane per workgroup");
static_assert(RCD_SLICES_MAX * SLICE_SAMPLES <= 1 << J_BITS, "samples of the largest class that is cut into slices");

// High words of keys: a candidate's is above KEY_LIVE (of -1e299: 0x01FCE302); KEY_UNKNOWN where a list of the best ends.
constexpr unsigned KEY_LIVE = 0x02000000u, KEY_UNKNOWN = 0xFFFFFFFFu;

template <typename S> struct SliceShared {
    Slot slots[S::KM][2][4 * S::NW];         // per block and 16 lanes: the best candidate and the second
    Slot list[BM][BM];                       // per block of this trip: the class's best, in order
    int listed[BM];                          // how many of them are known
    Entry stage[BM * S::NW][POST - 1];
    int count[BM * S::NW];                   // entries of wave w's part of pick u's list
    Entry mine[POST];                        // what travels in my post
    Entry entries[ENTRIES];                  // the lists that are applied here, end to end
    int len[BM][RCD_SLICES_MAX], at[BM][RCD_SLICES_MAX];     // of workgroup i's segments: the lengths, and where they go
    int fetch[RCD_SLICES_MAX];                   // workgroup i's segments did not travel in its post
    int nd[BM];                              // the lists' lengths
    int kept, sure, any_long;                // bit u: list u is applied here; picks that fit into this trip
    int ok[BM];
    int guesses, ahead;                      // how the guesses went (guess_after()), and the most of a trip
};

// Every row of 16 lanes puts its best candidate and its second for block k into the slots.  They stay from trip to trip: a wave
// writes a block's anew when one of the two was taken or has lost gain (mine: the blocks for which this lane holds one of the two).
// Decided by the high words of the keys; a tie there takes the long way.
template <typename S>
__device__ __forceinline__ void row_candidates(const double (&G)[S::KM][S::P], int k, const SlicePlace<S> &pl, Slot (*slots)[4 * S::NW],
                                               unsigned &mine)
{
    double t[S::P];
    resident::at_index<0, S::KM>(k, [&](auto kc) {
#pragma unroll
        for (int i = 0; i < S::P; ++i) t[i] = G[decltype(kc)::value][i];
    });
    mine &= ~(1u << k);
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        double s[S::P];
#pragma unroll
        for (int i = 0; i < S::P; ++i) s[i] = t[i];
#pragma unroll
        for (int w = 1; w < S::P; w *= 2)
#pragma unroll
            for (int i = 0; i + w < S::P; i += 2 * w) s[i] = resident::max_f64(s[i], s[i + w]);
        // the lowest of the lane's samples that has it: pieces ascending, then the lane's two
        int at = 0;
#pragma unroll
        for (int i = S::P - 1; i >= 1; --i) at = t[i] == s[0] ? i : at;
        at = t[0] == s[0] ? 0 : at;
        unsigned hi, lo;
        resident::key_words(s[0], hi, lo);
        const int v = (int)pl.v0 + (at >> 1) * 128 + (at & 1);
        bool win = hi == resident::row_max_u32(hi);
        if (__popcll(__ballot(win)) != 4) {
            const unsigned low = resident::row_max_u32(win ? lo : 0u);
            win = win & (lo == low);
            const unsigned first = resident::row_max_u32(win ? ~(unsigned)v : 0u);
            win = win & (~(unsigned)v == first);
        }
        if (win) {
            slots[round][pl.wave * 4 + (pl.lane >> 4)] = Slot{hi, lo, v, 0};
            mine |= 1u << k;
        }
#pragma unroll
        for (int i = 0; i < S::P; ++i) t[i] = (win & (at == i)) ? INC_TAKEN : t[i];
    }
}

// ob[i]: the block that is i-th least in f of those with room (lowest index on ties), -1 where there are fewer.
template <int N> __device__ __forceinline__ void order_one_by_one(double f, int room, int lane, int (&ob)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        ob[i] = resident::choose_block(f, room);
        if ((lane & 15) == ob[i]) room = 0;
    }
}
// The same by counting, for every block, the blocks before it: no chain from one to the next.  Equal f take the long way.
// Blocks sit in the lanes 0 .. KM - 1 (those past K have no room).
template <int KM, int N> __device__ __forceinline__ void order_blocks(double f, int room, int lane, int (&ob)[N])
{
    using resident::dpp;
    unsigned hi, lo;
    resident::key_words(-f, hi, lo);
    hi = room <= 0 ? 0u : hi;
    lo = room <= 0 ? 0u : lo;
    const unsigned long long me = ((unsigned long long)hi << 32) | lo;
    int before = 0;
    unsigned long long equal = 0ull;
    auto against = [&](unsigned h, unsigned l) __attribute__((always_inline)) {
        const unsigned long long it = ((unsigned long long)h << 32) | l;
        before += it > me ? 1 : 0;
        equal |= __ballot(it == me);
    };
    auto quad = [&](unsigned h, unsigned l, bool self) __attribute__((always_inline)) {
        if (!self) against(h, l);
        against((unsigned)dpp<0xB1>((int)h), (unsigned)dpp<0xB1>((int)l));        // the lanes 1, 2, 3 away (exclusive or)
        against((unsigned)dpp<0x4E>((int)h), (unsigned)dpp<0x4E>((int)l));
        against((unsigned)dpp<0x1B>((int)h), (unsigned)dpp<0x1B>((int)l));
    };
    quad(hi, lo, true);
    if constexpr (KM > 4) quad((unsigned)dpp<0x141>((int)hi), (unsigned)dpp<0x141>((int)lo), false);     // 7 away, 6, 5, 4
    if constexpr (KM > 8) {
        const unsigned h = (unsigned)dpp<0x140>((int)hi), l = (unsigned)dpp<0x140>((int)lo);             // 15 away, 14, 13, 12
        quad(h, l, false);
        quad((unsigned)dpp<0x141>((int)h), (unsigned)dpp<0x141>((int)l), false);                         // 8 away, 9, 10, 11
    }
    const bool open = lane < KM && room > 0;
    if ((equal & __ballot(open)) != 0ull) {
        order_one_by_one(f, room, lane, ob);
        return;
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const unsigned long long it = __ballot(open && before == i);
        ob[i] = it ? (int)__builtin_ctzll(it) : -1;
    }
}

// A lane per candidate: the lane that holds the best (largest key, lowest sample on ties).
__device__ __forceinline__ int best_lane(unsigned hi, unsigned lo, int v)
{
    const unsigned top = wave_max_u32(hi);
    unsigned long long who = __ballot(hi == top);
    if (who & (who - 1ull)) {
        const unsigned low = wave_max_u32(hi == top ? lo : 0u);
        const unsigned first = wave_max_u32(hi == top && lo == low ? ~(unsigned)v : 0u);
        who = __ballot(hi == top && lo == low && ~(unsigned)v == first);
    }
    return (int)__builtin_ctzll(who);
}

// f(integral_constant u) for every pick of a trip
template <typename F> __device__ __forceinline__ void each_pick(F &&f)
{
    f(std::integral_constant<int, 0>{});
    f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{});
    f(std::integral_constant<int, 3>{});
    f(std::integral_constant<int, 4>{});
    f(std::integral_constant<int, 5>{});
    f(std::integral_constant<int, 6>{});
    f(std::integral_constant<int, 7>{});
}

__device__ __forceinline__ float max2(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

__device__ __forceinline__ double lane_double(double x, int l)
{
    const long long b = __double_as_longlong(x);
    return __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)(b >> 32), l) << 32) |
                                (unsigned)__builtin_amdgcn_readlane((int)b, l));
}

// inclusive sum over the lanes
__device__ __forceinline__ int wave_prefix(int x, int lane)
{
    x += resident::dpp<0x111>(x);
    x += resident::dpp<0x112>(x);
    x += resident::dpp<0x114>(x);
    x += resident::dpp<0x118>(x);
    const int r0 = __builtin_amdgcn_readlane(x, 15), r1 = __builtin_amdgcn_readlane(x, 31);
    const int r2 = __builtin_amdgcn_readlane(x, 47);
    return x + (lane >= 16 ? r0 : 0) + (lane >= 32 ? r1 : 0) + (lane >= 48 ? r2 : 0);
}

// two pieces of a slot, requested together
__device__ __forceinline__ void dev_load4x2(const int32_t *p, i32x4 &a, i32x4 &b)
{
    asm volatile("global_load_dwordx4 %0, %2, off sc1\n\t"
                 "global_load_dwordx4 %1, %2, off offset:16 sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(a), "=&v"(b)
                 : "v"(p)
                 : "memory");
}

__device__ __forceinline__ int32_t *slot_of(const MwExchange &x, int w)
{
    return x.banks + RCD_SLICE_INTS * w + POST_INTS * (x.epoch & 1u);
}
// The pieces first, first + 1, ... of this workgroup's post, one per lane from lane 0 on.  One wave.
__device__ __forceinline__ void put(const MwExchange &x, int lane, int first, int pieces, int a, int b, int c)
{
    const unsigned piece = (unsigned)(first + lane);
    if (lane < pieces)
        dev_store4i(slot_of(x, x.w) + 4 * piece, a, b, c, (int)mw_tag(x.epoch + 0x01000000u * piece, (unsigned)a, (unsigned)b, (unsigned)c));
}
__device__ __forceinline__ bool fits(const MwExchange &x, int piece, const i32x4 &s)
{
    return (unsigned)s.w == mw_tag(x.epoch + 0x01000000u * (unsigned)piece, (unsigned)s.x, (unsigned)s.y, (unsigned)s.z);
}

// Looks at posts (`look` asks for what it needs and says whether all of it is there) until they have come.  One wave.  False when
// the bounded wait has run out or the flag is up.
template <typename F> __device__ __forceinline__ bool wait_for(const MwExchange &x, F &&look)
{
    for (int it = 1;; ++it) {
        if (__all(look())) return true;
        // (now and then: the flag is a trip of its own between two looks at the posts)
        if ((it & 15) == 0 && __hip_atomic_load(x.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2) return false;
        if ((it & 15) <= 1) {
            if (wall_clock64() > x.deadline) {
                __hip_atomic_store(x.abort_flag, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return false;
            }
        }
    }
}

// N candidates of a block, this workgroup's best in order (lane g of `p` holds the g-th), to everybody, as pieces from `first` on;
// then the class's best, in order and as far as they are known, into `list`: at most `need`.  Returns how many, -1 when the wait
// has run out.  One wave.
template <int N>
__device__ __forceinline__ int class_best(const MwExchange &x, int lane, int first, const Slot &p, int need, Slot *list)
{
    static_assert(N == 2 || N == 4 || N == 8, "loads");
    i32x4 s[N];                                  // lane w: workgroup w's
    if (x.W > 1) {
        put(x, lane, first, N, (int)p.hi, (int)p.lo, p.v);
        const int32_t *src = slot_of(x, lane) + 4 * first;
        const bool ok = wait_for(x, [&]() {
            bool good = true;
            if (lane < x.W) {
                if constexpr (N == 2) dev_load4x2(src, s[0], s[1]);
                else dev_load4x4(src, s[0], s[1], s[2], s[3]);
                if constexpr (N == 8) dev_load4x4(src + 16, s[4], s[5], s[6], s[7]);
#pragma unroll
                for (int g = 0; g < N; ++g) good = good && fits(x, first + g, s[g]);
            }
            return good;
        });
        if (!ok) return -1;
    } else {
#pragma unroll
        for (int g = 0; g < N; ++g)
            s[g] = (i32x4){__builtin_amdgcn_readlane((int)p.hi, g), __builtin_amdgcn_readlane((int)p.lo, g), __builtin_amdgcn_readlane(p.v, g), 0};
    }
#pragma unroll
    for (int g = 0; g < N; ++g) s[g].x = lane < x.W ? s[g].x : 0;       // (the key 0 is below every number's)
    int n = 0;
    for (; n < need; ++n) {
        const int src = best_lane((unsigned)s[0].x, (unsigned)s[0].y, s[0].z);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane(s[0].x, src);
        if (hi - KEY_LIVE >= KEY_UNKNOWN - KEY_LIVE) break;
        if (lane == src) {
            list[n] = Slot{hi, (unsigned)s[0].y, s[0].z, 0};
#pragma unroll
            for (int g = 0; g + 1 < N; ++g) s[g] = s[g + 1];
            s[N - 1].x = (int)KEY_UNKNOWN;       // behind a workgroup's last nothing is known
        }
    }
    return n;
}

} // namespace sliced

// Greedy steps of the incremental-gain route, W workgroups per class (wgmap[b] = class, index among the class's workgroups,
// their count), at most max_steps of them.  Lists of more than `small` rows are left to the update launch, as
// rcd_k_inc_steps_mw leaves them (segments of the workgroups, one after the other).
template <typename S>
__global__ void __launch_bounds__(S::NT)
rcd_k_inc_steps_sliced(RcdClass *__restrict__ classes, RcdPlan *__restrict__ plans, const RcdWg *__restrict__ wgmap,
                       int max_steps, int small_bytes, unsigned epoch0, long long spin_ticks)
{
    using namespace sliced;
    constexpr int NW = S::NW, Q = S::Q, P = S::P;
    static_assert(NW == BM && BM == 8, "a wave per block, a lane per pick and wave");
    __shared__ __attribute__((aligned(16))) SliceShared<S> sh;
    const RcdWg wg = wgmap[blockIdx.x];
    RcdClass &st = classes[__builtin_amdgcn_readfirstlane(wg.cls)];
    if ((st.done | plans[0].bad) != 0) return;      // (the same in all of a class's workgroups, or the waits end by the flag)
    const long long tick0 = wall_clock64();
    const int w = __builtin_amdgcn_readfirstlane(wg.w), W = __builtin_amdgcn_readfirstlane(wg.W);
    const int K = __builtin_amdgcn_readfirstlane(st.K), n = __builtin_amdgcn_readfirstlane(st.n);
    const int ld = __builtin_amdgcn_readfirstlane(st.ld), mwseg = __builtin_amdgcn_readfirstlane(st.mwseg);
    const gcf32 M = (gcf32)mw_uniform(st.M);
    const gf32 cur_all = (gf32)mw_uniform(st.cur);
    // what is needed now and then is read from the descriptor then: scalar registers are short
    auto rarely = [&]() {
        const RcdClass *again = &st;
        asm volatile("" : "+s"(again));
        return again;
    };
    int32_t *mwbuf = mw_uniform(st.mwbuf);
    const int s0 = min(w * mwseg, ld), s1 = min(s0 + mwseg, ld);
    const int small = (int)max(4ll, min((long long)INC_SMALL, (long long)small_bytes * W / ((long long)ld * 4)));
    SlicePlace<S> pl;
    pl.init(s0, s1);
    const int lane = pl.lane;
    const unsigned long long below = (1ull << lane) - 1ull;
    Run r;
    resident::load_run(r, st, max_steps);
    double G[S::KM][P];
    resident::load_gains<S>(G, inc_gains(st), K, n, ld, pl);
    MwExchange x;
    x.banks = mw_uniform(inc_slices(st));
    x.abort_flag = &plans[0].bad;
    x.W = W;
    x.w = w;
    x.epoch = epoch0 + 1;
    x.deadline = tick0 + spin_ticks;
    if (S::LEARN && threadIdx.x == 0) {
        const int word = guess_loaded(mwbuf[MW_SLOT]);       // (this loop's posts are in inc_slices())
        sh.guesses = word;
        sh.ahead = guesses_ahead(word);
    }
    bool alive = true;
    long long entries = 0, sweeps = 0;
    // everyone has read the descriptor before anyone may write it back
    if (W > 1) {
        __syncthreads();
        if (pl.wave == 0) {
            put(x, lane, 0, 1, 0, 0, 0);
            const bool ok = wait_for(x, [&]() { return lane >= W || fits(x, 0, dev_load4(slot_of(x, lane))); });
            if (lane == 0) sh.ok[0] = ok;
        }
        lds_barrier();
        alive = sh.ok[0] != 0;
    }
    auto write_held = [&]() {
        const RcdClass *c = rarely();
        if (w == 0) resident::write_outputs<S>(r, c->assign_out, c->order_out, c->out_index, pl);
        r.held = 0;
    };
    int ob[BM];                                  // the least blocks, in order
    order_blocks<S::KM>(r.f, r.room, lane, ob);
    unsigned calm = 0;                           // bit k: block k's last list was applied here, its next pick's may be guessed to be
    int span = BM;                               // the blocks a trip looks at, at most
    unsigned dirty = 0xFFFFu, mine = 0;          // bit k: this wave's entries of block k in the slots are not current; see row_candidates()
    while (alive) {
        if (r.t >= r.total || ob[0] < 0) { r.done = 1; break; }
        if (r.t - r.t0 >= r.max_steps) { r.stop = 1; break; }
        if (!((r.valid >> ob[0]) & 1u)) break;
        // ---- the blocks: the u-th pick goes to one of the u least (f never falls)
        const int most = min(min(r.total - r.t, r.max_steps - (r.t - r.t0)), BM);
        int nb = 0, pos = -1, order = -1;        // how many; lane k: block k's place among them; lane i: the i-th of them
#pragma unroll
        for (int i = 0; i < BM; ++i)
            if (nb == i && i < min(most, span) && ob[i] >= 0 && ((r.valid >> (ob[i] & 15)) & 1u)) {
                nb = i + 1;
                pos = (lane & 15) == ob[i] ? i : pos;
                order = lane == i ? ob[i] : order;
            }
        // ---- candidates of this slice
#pragma unroll
        for (int i = 0; i < BM; ++i)
            if (i < nb && ((dirty >> ob[i]) & 1u)) {
                row_candidates<S>(G, ob[i], pl, sh.slots[ob[i]], mine);
                dirty &= ~(1u << ob[i]);
            }
        lds_barrier();
        x.epoch += 1;
        if (pl.wave < nb) {
            // a wave per block: this workgroup's best, and with everybody's the class's
            const int k = __builtin_amdgcn_readlane(order, pl.wave);
            const int ahead = S::LEARN ? __builtin_amdgcn_readfirstlane(sh.ahead) : GUESS_MOST;
            // how many of the class's are wanted (without guesses only what other blocks' picks take is to be made up for) and posted
            const int need = ahead == 0 ? min(nb, 3) : nb == 1 ? 1 + ahead : nb == 2 ? 6 : nb <= 4 ? 4 : 3;
            const int share = nb > 4 || need <= 2 ? 2 : nb > 2 || need <= 4 ? 4 : 8;
            Slot a = sh.slots[k][lane >> 5][lane & 31], p = Slot{KEY_UNKNOWN, 0u, -1, 0};
            for (int g = 0; g < share; ++g) {
                const int src = best_lane(a.hi, a.lo, a.v);
                const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)a.hi, src), lo = (unsigned)__builtin_amdgcn_readlane((int)a.lo, src);
                const int v = __builtin_amdgcn_readlane(a.v, src);
                if (lane == g) p = Slot{hi, lo, v, 0};
                if (src >= 32) break;            // (a row's second is gone: its third is not known)
                if (lane == src) a.hi = 0u;
            }
            int got;
            if (share == 2) got = class_best<2>(x, lane, pl.wave * 2, p, need, sh.list[pl.wave]);
            else if (share == 4) got = class_best<4>(x, lane, pl.wave * 4, p, need, sh.list[pl.wave]);
            else got = class_best<8>(x, lane, pl.wave * 8, p, need, sh.list[pl.wave]);
            if (lane == 0) {
                sh.listed[pl.wave] = got;
                sh.ok[pl.wave] = got >= 0;
            }
        }
        lds_barrier();
        if (__ballot(lane < nb && sh.ok[lane & (BM - 1)] == 0) != 0ull) { alive = false; break; }

        // ---- the picks, on the gains as they are (every wave of every workgroup alike): lane 8 i + g holds the g-th best candidate
        //      of the i-th block
        int B = 0;
        int of_j = 0, of_v = 0, of_same = 0;     // lane u: pick u's block, its sample, the picks before it for the same block
        double of_gain = 0.0;
        unsigned guess = 0;                      // the picks that have such
        unsigned picked = 0;                     // lane k: the picks for block k
        auto pj = [&](int u) { return __builtin_amdgcn_readlane(of_j, u); };
        auto pv = [&](int u) { return __builtin_amdgcn_readlane(of_v, u); };
        auto same = [&](int u) { return (unsigned)__builtin_amdgcn_readlane(of_same, u); };
        f32x2 mp[BM][Q], two[2][Q];              // their rows, and the coverage that two of them are held against
        auto ask_cover = [&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            if (u < B) {
                const gcf32 row = (gcf32)(cur_all + (size_t)pj(u) * ld);
#pragma unroll
                for (int q = 0; q < Q; ++q) two[u & 1][q] = pl.at(row, q);
            }
        };
        int next[BM];
        double ft = r.f;                         // f and room with the picks made
        int roomt = r.room;
        {
            const Slot cand = sh.list[lane >> 3][lane & 7];
            int ahead = S::LEARN ? __builtin_amdgcn_readfirstlane(sh.ahead) : GUESS_MOST;
            unsigned long long avail = __ballot((lane >> 3) < nb && (lane & 7) < sh.listed[lane >> 3]);
            int at = 0, js = ob[0], turn = 1;    // the next of the blocks in order that has no pick yet
            unsigned before = 0;                 // the picks for block js
            double least = INFINITY;             // f among the blocks that have one
#pragma unroll
            for (int u = 0; u < BM; ++u)
                if (B == u && u < most && js >= 0) {
                    const unsigned some = at >= 0 ? (unsigned)(avail >> (at & 63)) & 0xFFu : 0u;
                    if (some != 0u && (before == 0u || (((calm >> js) & 1u) && ahead > 0))) {
                        const int src = at + (int)__builtin_ctz(some);
                        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)cand.hi, src), lo = (unsigned)__builtin_amdgcn_readlane((int)cand.lo, src);
                        const double gain = inc_value(((unsigned long long)hi << 32) | lo);
                        const int vstar = __builtin_amdgcn_readlane(cand.v, src);
                        const gcf32 row = M + (size_t)(unsigned)vstar * (unsigned)ld;
#pragma unroll
                        for (int q = 0; q < Q; ++q) mp[u][q] = pl.at(row, q);
                        of_j = lane == u ? js : of_j;
                        of_v = lane == u ? vstar : of_v;
                        of_same = lane == u ? (int)before : of_same;
                        of_gain = lane == u ? gain : of_gain;
                        guess |= before ? 1u << u : 0u;
                        if constexpr (S::LEARN) ahead -= before ? 1 : 0;
                        B = u + 1;
                        const bool it = (lane & 15) == js;
                        const double more = ft + gain;
                        ft = it ? more : ft;
                        roomt = it ? roomt - 1 : roomt;
                        picked = it ? picked | 1u << u : picked;
                        avail &= ~__ballot(cand.v == vstar);
                        if (u + 1 < BM) {
                            // the next block: the next in order, unless one that has a pick is at most that much
                            least = fmin(least, lane_double(ft, js));
                            const int k = __builtin_amdgcn_readlane(order, turn);
                            if (turn < nb && __ballot(!(lane_double(r.f, k & 15) < least)) == 0ull) {
                                js = k;
                                at = 8 * turn;
                                before = 0;
                                ++turn;
                            } else {
                                js = resident::choose_block(ft, roomt);
                                at = 8 * __builtin_amdgcn_readlane(pos, js & 15);
                                before = (unsigned)__builtin_amdgcn_readlane((int)picked, js & 15);
                                turn = BM;
                            }
                        }
                    }
                }
            if (B == 0) { r.done = 1; break; }   // no candidate left (cannot happen while t < total <= n)
            ask_cover(std::integral_constant<int, 0>{});
            ask_cover(std::integral_constant<int, 1>{});
            // (while these are on their way: the blocks' order after the picks)
            order_blocks<S::KM>(ft, roomt, lane, next);
            __builtin_amdgcn_sched_barrier(0);
        }

        // ---- coverage: the j of this slice with S(j, v*) > cur_k(j), ascending
        // f(position in the wave's part of the list, j, old, new) for every entry
        auto each_entry = [&](const f32x2 (&row)[Q], const f32x2 (&c)[Q], auto &&f) {
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q < pl.nq) {
                    const bool ch0 = row[q].x > c[q].x, ch1 = row[q].y > c[q].y;
                    const unsigned long long b0 = __ballot(ch0), b1 = __ballot(ch1);
                    if ((b0 | b1) != 0ull) {
                        const int pos = cnt + __popcll(b0 & below) + __popcll(b1 & below);
                        const int v = (int)pl.v0 + 128 * q;
                        if (ch0) f(pos, v, c[q].x, row[q].x);
                        if (ch1) f(pos + (ch0 ? 1 : 0), v + 1, c[q].y, row[q].y);
                        cnt += __popcll(b0) + __popcll(b1);
                    }
                }
            return cnt;
        };
        each_pick([&](auto uc) {
            constexpr int u = decltype(uc)::value;
            int cnt = 0;
            if (u < B) {
                f32x2 (&c)[Q] = two[u & 1];
                if (u > 0 && ((guess >> u) & 1u)) {
                    // (what the block's picks before it leave)
                    const unsigned before = same(u);
#pragma unroll
                    for (int p = 0; p < u; ++p)
                        if ((before >> p) & 1u) {
#pragma unroll
                            for (int q = 0; q < Q; ++q) c[q] = (f32x2){max2(c[q].x, mp[p][q].x), max2(c[q].y, mp[p][q].y)};
                        }
                }
                Entry *held = sh.stage[u * NW + pl.wave];
                cnt = each_entry(mp[u], c, [&](int pos, int j, float o, float nw) {
                    if (pos < POST - 1) held[pos] = Entry{j, o, nw, 0};
                });
            }
            if constexpr (u + 2 < BM) ask_cover(std::integral_constant<int, u + 2>{});
            if (lane == 0) sh.count[u * NW + pl.wave] = cnt;
        });
        lds_barrier();

        // ---- the lists: lane u NW + i holds the length of wave i's part for pick u
        const int found = sh.count[lane];
        const int incl = wave_prefix(found, lane);
        const int all = __builtin_amdgcn_readlane(incl, 63);
        // the segments' lengths, and this wave's place in them
        auto before = [&](int u) { return u > 0 ? __builtin_amdgcn_readlane(incl, u * NW - 1) : 0; };
        auto len = [&](int u) { return __builtin_amdgcn_readlane(incl, u * NW + NW - 1) - before(u); };
        auto base = [&](int u) { return __builtin_amdgcn_readlane(incl - found, u * NW + pl.wave) - before(u); };
        // Pick u's part of this wave to memory: its segment and, where asked for, the new coverage.  (Coverage in memory is what the
        // pick found: nothing has been written for the block, or only for the picks before it.)
        auto write_segment = [&](int u, bool coverage) {
            const int k = pj(u);
            f32x2 row[Q], c[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                row[q] = pl.at(M + (size_t)pv(u) * ld, q);
                c[q] = pl.at((gcf32)(cur_all + (size_t)k * ld), q);
            }
            const size_t at = (size_t)k * ld + s0 + base(u);
            const RcdClass *d = rarely();
            const gi32 dlist = (gi32)inc_dlist(*d);
            const gf32 dold = (gf32)inc_dold(*d), dnew = (gf32)inc_dnew(*d);
            each_entry(row, c, [&](int pos, int j, float o, float nw) {
                dev_store(dlist + at + pos, j);
                dev_store(dold + at + pos, o);
                dev_store(dnew + at + pos, nw);
                if (coverage) *off<float>(cur_all + (size_t)k * ld, (unsigned)j * 4u) = nw;
            });
        };
        // Too many entries for the post: they go to memory.  (There is one segment per block, so of a block's picks the first one's:
        // a guess behind it does not hold then.)
        const bool in_memory = all > POST - 1;
        if (in_memory) {
            for (int u = 0; u < B; ++u)
                if (!((guess >> u) & 1u)) write_segment(u, false);
            wait_for_my_stores();
            lds_barrier();
        }
        x.epoch += 1;
        if (pl.wave == 0) {
            if (!in_memory) {
                const int start = __builtin_amdgcn_ds_bpermute(4 * (lane & ~(NW - 1)), incl - found);      // of the pick's
                for (int g = 0; g < found; ++g) {
                    Entry e = sh.stage[lane][g];
                    e.j = entry_word(e.j, lane / NW, incl - found + g - start);
                    sh.mine[1 + incl - found + g] = e;
                }
            }
            __builtin_amdgcn_wave_barrier();
            int a = (int)post_word0(len(0), len(1), len(2)), b = (int)post_word1(len(2), len(3), len(4), len(5));
            int d = (int)post_word2(len(5), len(6), len(7));
            if (lane > 0 && lane < POST) {
                const Entry e = sh.mine[lane];
                a = e.j;
                b = __float_as_int(e.o);
                d = __float_as_int(e.n);
            }
            const int pieces = in_memory ? 1 : 1 + all;
            i32x4 s[4];
            bool ok = true;
#pragma unroll
            for (int g = 0; g < 4; ++g) s[g] = (i32x4){0, 0, 0, 0};
            auto lengths = [&](int (&l)[BM]) {
#pragma unroll
                for (int u = 0; u < BM; ++u) l[u] = post_length(u, (unsigned)s[0].x, (unsigned)s[0].y, (unsigned)s[0].z);
            };
            int l[BM], more = 0;                 // a workgroup per lane: its segments' lengths, the entries in its post
            if (W > 1) {
                put(x, lane, 0, pieces, a, b, d);
                ok = wait_for(x, [&]() {
                    bool good = true;
                    if (lane < W) {
                        dev_load4x4(slot_of(x, lane), s[0], s[1], s[2], s[3]);
                        good = fits(x, 0, s[0]);
                        lengths(l);
                        more = entries_in_post(l[0] + l[1] + l[2] + l[3] + l[4] + l[5] + l[6] + l[7]);
#pragma unroll
                        for (int g = 1; g < 4; ++g) good = good && (g > more || fits(x, g, s[g]));
                    }
                    return good;
                });
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    if (lane == 0) s[g] = (i32x4){__builtin_amdgcn_readlane(a, g), __builtin_amdgcn_readlane(b, g), __builtin_amdgcn_readlane(d, g), 0};
                more = lane == 0 && !in_memory ? all : 0;
            }
            lengths(l);
#pragma unroll
            for (int u = 0; u < BM; ++u) l[u] = believed(ok && lane < W, l[u]);
            more = believed(ok, more);
            // places of the segments in the lists; a list that is too long stays so if its segments' lengths are cut here
            int kept = 0, total = 0, sure = 0;
            int nd[BM], ahead[BM];
            bool room = true;
#pragma unroll
            for (int u = 0; u < BM; u += 2) {
                const int x0 = min(l[u], 1023), x1 = min(l[u + 1], 1023), both = x0 | x1 << 16;
                const int in = wave_prefix(both, lane), sum = __builtin_amdgcn_readlane(in, 63);
                nd[u] = sum & 0xFFFF;
                nd[u + 1] = (int)((unsigned)sum >> 16);
                ahead[u] = (in - both) & 0xFFFF;
                ahead[u + 1] = (int)((unsigned)(in - both) >> 16);
            }
#pragma unroll
            for (int u = 0; u < BM; ++u) {
                const int n_u = nd[u] > small ? 0 : nd[u];
                room = room && u < B && total + n_u <= ENTRIES;
                if (room) {
                    sure = u + 1;
                    if (nd[u] <= small) kept |= 1 << u;
                    sh.at[u][lane] = total + ahead[u];
                    total += n_u;
                }
            }
            if (__ballot(l[0] > 1023 || l[1] > 1023 || l[2] > 1023 || l[3] > 1023 || l[4] > 1023 || l[5] > 1023 || l[6] > 1023 ||
                         l[7] > 1023) != 0ull) {
#pragma unroll
                for (int u = 0; u < BM; ++u) nd[u] = __builtin_amdgcn_readlane(wave_prefix(l[u], lane), 63);
            }
            if (lane == 0) {
#pragma unroll
                for (int u = 0; u < BM; ++u) sh.nd[u] = nd[u];
                sh.kept = kept;
                sh.sure = sure;
            }
            __builtin_amdgcn_wave_barrier();
            auto place = [&](const i32x4 &e, int g) {
                const int u = entry_pick(e.x), i = entry_place(e.x);
                if (g <= more && ((kept >> u) & 1)) {
                    const int at = sh.at[u][lane] + i;
                    sh.entries[at] = Entry{e.x & ((1 << (J_BITS + 3)) - 1), __int_as_float(e.y), __int_as_float(e.z), 0};
                }
            };
#pragma unroll
            for (int g = 1; g < 4; ++g) place(s[g], g);
            // entries beyond the first three of a post
            for (int first = 4; ok && __ballot(more >= first) != 0ull; first += 4) {
                if (W > 1) {
                    ok = wait_for(x, [&]() {
                        bool good = true;
                        if (more >= first) {
                            dev_load4x4(slot_of(x, lane) + 4 * first, s[0], s[1], s[2], s[3]);
#pragma unroll
                            for (int g = 0; g < 4; ++g) good = good && (first + g > more || fits(x, first + g, s[g]));
                        }
                        return good;
                    });
                } else {
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        if (lane == 0)
                            s[g] = (i32x4){__builtin_amdgcn_readlane(a, first + g), __builtin_amdgcn_readlane(b, first + g),
                                           __builtin_amdgcn_readlane(d, first + g), 0};
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) place(s[g], first + g);
            }
            // segments that did not travel in the posts
            bool fetch = false;
#pragma unroll
            for (int u = 0; u < BM; ++u) fetch = fetch || (l[u] > 0 && ((kept >> u) & 1));
            fetch = fetch && more == 0 && lane < W;
            const bool lng = __ballot(fetch) != 0ull;
            if (lng) {
                sh.fetch[lane] = fetch;
#pragma unroll
                for (int u = 0; u < BM; ++u) sh.len[u][lane] = (kept >> u) & 1 ? l[u] : 0;
            }
            if (lane == 0) {
                sh.any_long = lng;
                sh.ok[0] = ok;
            }
        }
        lds_barrier();
        if (sh.ok[0] == 0) { alive = false; break; }
        const int kept = __builtin_amdgcn_readfirstlane(sh.kept);
        const bool any_long = __builtin_amdgcn_readfirstlane(sh.any_long) != 0;
        // the picks below `sure` hold, so far: a guess does not behind a list that is left to the update launch, or where segments are
        // in memory
        int sure = __builtin_amdgcn_readfirstlane(sh.sure);
        if (guess) {
#pragma unroll
            for (int u = BM - 1; u >= 1; --u)
                if (same(u) != 0u && ((same(u) & ~(unsigned)kept) != 0u || any_long)) sure = min(sure, u);
        }
        const int lengths = sh.nd[lane & (BM - 1)];
        auto nd = [&](int u) { return __builtin_amdgcn_readlane(lengths, u); };
        int total = 0;
#pragma unroll
        for (int u = 0; u < BM; ++u) total += u < sure && ((kept >> u) & 1) ? nd(u) : 0;
        if (any_long) {
            // a wave per workgroup's segments
            const RcdClass *d = rarely();
            const gi32 dlist = (gi32)inc_dlist(*d);
            const gf32 dold = (gf32)inc_dold(*d), dnew = (gf32)inc_dnew(*d);
            for (int i = pl.wave; i < W; i += NW) {
                if (sh.fetch[i] == 0) continue;
                each_pick([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    if (u >= sure) return;
                    const int n_u = sh.len[u][i], to = sh.at[u][i];
                    const size_t from = (size_t)pj(u) * ld + (size_t)i * mwseg;
                    for (int e = lane; e < n_u; e += 64)
                        sh.entries[to + e] = Entry{dev_load(dlist + from + e) | u << J_BITS, dev_load(dold + from + e), dev_load(dnew + from + e), 0};
                });
            }
            lds_barrier();
        }

        // ---- gains: the lists' terms, all lists end to end, added up per pick in list order, then onto the block's gains
        {
            double acc[P];
            int of = -1;                         // pick the sums are for
            unsigned long long touched = 0ull;   // lanes that have a term
            auto flush = [&]() {
                if (touched == 0ull) return;
                int k = pj(0);
#pragma unroll
                for (int u = 1; u < BM; ++u) k = of == u ? pj(u) : k;
                resident::update_at_index<0, S::KM>(k, [&](auto kc) {
#pragma unroll
                    for (int i = 0; i < P; ++i) G[decltype(kc)::value][i] += acc[i];
                });
                if ((touched & __ballot((mine >> k) & 1u)) != 0ull) dirty |= 1u << k;
            };
            constexpr int U = S::ROWS;           // rows in flight
            for (int first = 0; first < total; first += 64) {
                const Entry en = sh.entries[min(first + lane, total - 1)];
                const int there = min(64, total - first), j = entry_sample(en.j), pick = en.j >> J_BITS;
                // U rows at a time, the next ones under way; behind the end the last one again
                f32x2 m[2][U][Q];
                auto ask = [&](f32x2 (&rows)[U][Q], int e0) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < U; ++i) {
                        const gcf32 row = M + (size_t)(unsigned)__builtin_amdgcn_readlane(j, min(e0 + i, there - 1)) * (unsigned)ld;
#pragma unroll
                        for (int q = 0; q < Q; ++q) rows[i][q] = pl.at(row, q);
                    }
                };
                // Which of the rows have a sample nearer to j than j's old coverage (late in a run few have one in a wave), and these
                // rows' terms.
                int here = there;
                auto use = [&](const f32x2 (&rows)[U][Q], int e0) __attribute__((always_inline)) {
                    unsigned hit = 0;
#pragma unroll
                    for (int i = 0; i < U; ++i) {
                        float far = max2(rows[i][0].x, rows[i][0].y);
#pragma unroll
                        for (int q = 1; q < Q; ++q) far = resident::max3(rows[i][q].x, rows[i][q].y, far);
                        hit |= (__ballot(far > inc_lane_value(en.o, (e0 + i) & 63)) != 0ull ? 1u : 0u) << i;
                    }
                    if (here - e0 < U) hit &= (1u << (here - e0)) - 1u;
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        if ((hit >> i) & 1u) {
                            const int u = __builtin_amdgcn_readlane(pick, e0 + i);
                            if (u != of) {
                                flush();
                                of = u;
                                touched = 0ull;
#pragma unroll
                                for (int a = 0; a < P; ++a) acc[a] = 0.0;
                            }
                            const float cn = inc_lane_value(en.n, e0 + i), co = inc_lane_value(en.o, e0 + i);
                            bool any = false;
#pragma unroll
                            for (int q = 0; q < Q; ++q) {
                                any |= (rows[i][q].x > co) | (rows[i][q].y > co);
                                acc[2 * q] += inc_term(rows[i][q].x, cn, co);
                                acc[2 * q + 1] += inc_term(rows[i][q].y, cn, co);
                            }
                            touched |= __ballot(any);
                        }
                };
                // a guess whose similarity to an entry of the block's earlier picks is above the old coverage has lost gain
                float near[BM];
                if (guess) {
                    const gcf32 row = M + (size_t)j * ld;
#pragma unroll
                    for (int u = 1; u < BM; ++u)
                        if ((guess >> u) & 1u) near[u] = row[pv(u)];
                }
                ask(m[0], 0);
                if (there > U) ask(m[1], U);
                if (guess) {
#pragma unroll
                    for (int u = BM - 1; u >= 1; --u)
                        if (u < sure && ((guess >> u) & 1u) && __ballot(lane < there && ((same(u) >> pick) & 1u) && near[u] > en.o) != 0ull) sure = u;
                    here = __popcll(__ballot(lane < there && pick < sure));
                }
                for (int e0 = 0; e0 < here; e0 += 2 * U) {
                    use(m[0], e0);
                    if (e0 + U >= here) break;
                    if (e0 + 2 * U < here) ask(m[0], e0 + 2 * U);
                    use(m[1], e0 + U);
                    if (e0 + 3 * U < here) ask(m[1], e0 + 3 * U);
                }
                // the new coverage of this wave's samples (a block that was picked again: in the order of the picks)
                int k = pj(0);
#pragma unroll
                for (int u = 1; u < BM; ++u) k = pick == u ? pj(u) : k;
                const bool write = lane < here && (unsigned)(j - pl.first) < (unsigned)min(pl.nq * 128, S::WAVE);
                float RCD_GLOBAL *place = cur_all + (size_t)k * ld + j;
                if (!guess) {
                    if (write) *place = en.n;
                } else {
                    for (int u = 0; u < sure; ++u)
                        if (write && pick == u) *place = en.n;
                }
                if (here < there) break;         // the rest is of picks that do not hold
            }
            flush();
        }

        // ---- the picks that hold; the new coverage of this slice, and what is left to the update launch
        if (sure < B) {
            ft = r.f;
            roomt = r.room;
#pragma unroll
            for (int u = 0; u < BM; ++u)
                if (u < sure && (lane & 15) == pj(u)) {
                    ft += lane_double(of_gain, u);
                    roomt -= 1;
                }
            order_blocks<S::KM>(ft, roomt, lane, next);
        }
        r.f = ft;
        r.room = roomt;
#pragma unroll
        for (int u = 0; u < BM; ++u) ob[u] = next[u];
        {
            const bool it = lane >= r.held && lane < r.held + sure;
            const int j = __builtin_amdgcn_ds_bpermute(4 * (lane - r.held), of_j), v = __builtin_amdgcn_ds_bpermute(4 * (lane - r.held), of_v);
            r.held_j = it ? j : r.held_j;
            r.held_v = it ? v : r.held_v;
        }
        entries += lane < sure ? lengths : 0;
        // the samples of this wave among the picks
        for (unsigned long long it = __ballot(lane < sure && (unsigned)(of_v - pl.first) < (unsigned)S::WAVE); it; it &= it - 1ull) {
            const int v = pv((int)__builtin_ctzll(it));
            resident::strike<S>(G, v, pl.first, lane);
            dirty |= (unsigned)__builtin_amdgcn_readlane((int)mine, ((v - pl.first) & 127) >> 1);
        }
        const unsigned all_sure = (1u << sure) - 1u;
        calm |= (unsigned)__ballot(lane < 16 && (picked & (unsigned)kept & all_sure) != 0u);
        if (S::LEARN && threadIdx.x == 0) {
            // (everyone has read these two, and reads them again behind a barrier)
            const int word = guess_after(sh.guesses, __popc(guess & all_sure), ((guess >> sure) & 1u) != 0u);
            sh.guesses = word;
            sh.ahead = guesses_ahead(word);
        }
        span = blocks_after(__popcll(__ballot(lane < 16 && (picked & all_sure) != 0u)), BM);
        for (unsigned left = all_sure & ~(unsigned)kept; left; left &= left - 1u) {
            const int u = (int)__builtin_ctz(left), k = pj(u);
            write_segment(u, true);
            calm &= ~(1u << k);
            r.valid &= ~(1u << k);
            sweeps += 1;
            if (threadIdx.x == 0) {
                mwbuf[MW_PEND + k * RCD_SLICES_MAX + w] = len(u);
                if (w == 0) st.dcount[k] = nd(u);
            }
        }
        r.held += sure;
        r.nR -= sure;
        r.t += sure;
        if (r.held > 64 - BM) write_held();
    }
    if (!alive) return;          // a bounded wait ran out: plans[0].bad says so, nothing is written back
    write_held();
    if (!r.done) resident::store_gains<S>(G, inc_gains(st), K, ld, pl);
    if (w != 0) return;
    if (S::LEARN && threadIdx.x == 0) mwbuf[MW_SLOT] = guess_stored(sh.guesses);
#pragma unroll
    for (int i = 32; i >= 1; i >>= 1) entries += __shfl_xor(entries, i);
    resident::store_run(r, st, plans, entries * n, sweeps, true, wall_clock64() - tick0);
    const unsigned waiting = (unsigned)__ballot(lane < K && r.room > 0 && !((r.valid >> (lane & 15)) & 1u)) & 0xFFFFu;
    if (threadIdx.x == 0 && !r.done) {
        int nneed = 0;
        for (unsigned k = waiting; k; k &= k - 1u) st.need[nneed++] = (int)__builtin_ctz(k);
        st.nneed = nneed;
    }
}
