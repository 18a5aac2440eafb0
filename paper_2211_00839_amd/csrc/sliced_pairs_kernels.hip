// The loop of sliced_kernels.hip with two picks to a trip, for slices of more than 1024 samples with more than eight blocks: a
// slice's gains take 128 of a lane's 256 registers there, and the loop with up to eight picks to a trip has to keep too much of the
// rest in memory (16 classes of 20 000 samples and sixteen blocks 445 ms here, 499 there; 20 of them 508 and 578).
//   - The block after the one in turn is known before the pick: it is the least f among the others, unless the picked block stays
//     the least.  So the first post carries a workgroup's best candidate for the block in turn and its best two for the next one
//     (two, because the first pick may take the best), and when the guess holds, which every workgroup sees alike, one trip serves two
//     steps; so do the trips for the rows, the lists and the lists' rows.
// Picks, sums and ties are those of the other loops, in their order: the results are the same bits.
// The exchange itself (slots, tags, banks, bounded waits) is that of multi_wg_kernels.hip, and so is its area: at most
// RCD_MW_MAX workgroups to a class.
// Included by rcd_lib.hip after sliced_kernels.hip.
#include <hip/hip_runtime.h>
#include "rcd_state.h"

namespace pairs {

using resident::Entry;
using resident::Run;
using resident::Slot;
using resident::f32x2;
using resident::lds_barrier;
using resident::off;
using sliced::SlicePlace;
using sliced::best_lane;
using sliced::dev_load4x2;
using sliced::wave_prefix;

// 512 threads, Q pieces of two samples each, at most KM blocks, ROWS rows of the lists in flight.
template <int Q, int KM, int ROWS_> struct PairShape : resident::Shape<512, Q, KM> {
    static constexpr int ROWS = ROWS_;
};

template <typename S> struct PairShared {
    Slot slots[3][4 * S::NW];      // per 16 lanes: the best for the block in turn; the best and the second for the next
    Slot won[3];                   // the class's best of the block in turn, its best two of the next
    Entry stage[2 * S::NW][MW_INLINE];
    int count[2 * S::NW];          // entries of wave w's part of pick u's list
    Entry mine[MW_INLINE];         // what travels in my post
    Entry list[2 * INC_SMALL];     // the lists that are applied here, end to end
    int len[2][RCD_MW_MAX], pre[2][RCD_MW_MAX];   // what is applied here of workgroup i's segments, and where it goes
    int fetch[RCD_MW_MAX];         // workgroup i's segments did not travel in its post
    int nd[2];
    int ok[2], any_long;
};

// The best of a lane's samples: its key, and which of them it is (the first that has it).
template <typename S> struct LaneBest {
    unsigned hi, lo;
    int at;
    __device__ __forceinline__ void of(const double (&t)[S::P])
    {
        double s[S::P];
#pragma unroll
        for (int i = 0; i < S::P; ++i) s[i] = t[i];
#pragma unroll
        for (int w = 1; w < S::P; w *= 2)
#pragma unroll
            for (int i = 0; i + w < S::P; i += 2 * w) s[i] = resident::max_f64(s[i], s[i + w]);
        at = 0;
#pragma unroll
        for (int i = S::P - 1; i >= 1; --i) at = t[i] == s[0] ? i : at;
        at = t[0] == s[0] ? 0 : at;
        resident::key_words(s[0], hi, lo);
    }
    __device__ __forceinline__ int sample(const SlicePlace<S> &pl) const { return (int)pl.v0 + (at >> 1) * 128 + (at & 1); }
    // of the lanes of a row that tie in the high word, the one with the best candidate
    __device__ __forceinline__ bool settle(bool win, const SlicePlace<S> &pl) const
    {
        const unsigned low = resident::row_max_u32(win ? lo : 0u);
        win = win && lo == low;
        const unsigned v = ~(unsigned)sample(pl), first = resident::row_max_u32(win ? v : 0u);      // (by all lanes)
        return win && v == first;
    }
};

// Every row of 16 lanes puts its best candidate of the block in turn (t0) into slots[0] and, if there is a next block, its
// best two of that one (t1) into slots[1] and slots[2].  One chain without branches decides all three by the high words of
// the keys; a tie there takes the long way.
template <typename S>
__device__ __forceinline__ void row_candidates(const double (&t0)[S::P], const double (&t1)[S::P], bool two, const SlicePlace<S> &pl,
                                               Slot (*slots)[4 * S::NW])
{
    LaneBest<S> a, b, c;
    double t2[S::P];
    a.of(t0);
    bool wa = a.hi == resident::row_max_u32(a.hi), wb = false, wc = false;
    if (two) {
        b.of(t1);
        wb = b.hi == resident::row_max_u32(b.hi);
#pragma unroll
        for (int i = 0; i < S::P; ++i) t2[i] = wb && b.at == i ? INC_TAKEN : t1[i];
        c.of(t2);
        wc = c.hi == resident::row_max_u32(c.hi);
    }
    // (in a row that ties, every lane of the tie has given its best away: the second is found again)
    if (__popcll(__ballot(wa)) != 4) wa = a.settle(wa, pl);
    if (two && (__popcll(__ballot(wb)) != 4 || __popcll(__ballot(wc)) != 4)) {
        wb = b.settle(wb, pl);
#pragma unroll
        for (int i = 0; i < S::P; ++i) t2[i] = wb && b.at == i ? INC_TAKEN : t1[i];
        c.of(t2);
        wc = c.settle(c.hi == resident::row_max_u32(c.hi), pl);
    }
    const int row = pl.wave * 4 + (pl.lane >> 4);
    if (wa) slots[0][row] = Slot{a.hi, a.lo, a.sample(pl), 0};
    if (wb) slots[1][row] = Slot{b.hi, b.lo, b.sample(pl), 0};
    if (wc) slots[2][row] = Slot{c.hi, c.lo, c.sample(pl), 0};
}

// The pieces first, first + 1, ... of this workgroup's post, one per lane from lane 0 on.  One wave.
__device__ __forceinline__ void put(const MwExchange &x, int lane, int first, int pieces, int a, int b, int c)
{
    int32_t *slot = x.banks + (x.epoch & 1u) * (MW_SLOT_INTS * RCD_MW_MAX) + MW_SLOT_INTS * x.w;
    const unsigned piece = (unsigned)(first + lane);
    if (lane < pieces)
        dev_store4i(slot + 4 * piece, a, b, c, (int)mw_tag(x.epoch + 0x01000000u * piece, (unsigned)a, (unsigned)b, (unsigned)c));
}
__device__ __forceinline__ bool fits(const MwExchange &x, int piece, const i32x4 &s)
{
    return (unsigned)s.w == mw_tag(x.epoch + 0x01000000u * (unsigned)piece, (unsigned)s.x, (unsigned)s.y, (unsigned)s.z);
}

// Pieces of everybody's posts, a workgroup per lane: piece 0; pieces 1 and 2; or piece 0 = {length, length} and, where the
// lengths' sum is at most MW_INLINE, as many more.  One wave.  False when the bounded wait has run out or the flag is up.
enum { GET_FIRST = 0, GET_NEXT_TWO = 1, GET_LIST = 2 };
template <int KIND> __device__ __forceinline__ bool get(const MwExchange &x, int lane, i32x4 (&s)[4])
{
    const int32_t *slot = x.banks + (x.epoch & 1u) * (MW_SLOT_INTS * RCD_MW_MAX) + MW_SLOT_INTS * lane;
#pragma unroll
    for (int g = 0; g < 4; ++g) s[g] = (i32x4){0, 0, 0, 0};
    for (int it = 1;; ++it) {
        bool good = true;
        if (lane < x.W) {
            if constexpr (KIND == GET_FIRST) {
                s[0] = dev_load4(slot);
                good = fits(x, 0, s[0]);
            } else if constexpr (KIND == GET_NEXT_TWO) {
                dev_load4x2(slot + 4, s[0], s[1]);
                good = fits(x, 1, s[0]) && fits(x, 2, s[1]);
            } else {
                dev_load4x4(slot, s[0], s[1], s[2], s[3]);
                good = fits(x, 0, s[0]);
                const int more = s[0].x + s[0].y <= MW_INLINE ? s[0].x + s[0].y : 0;
#pragma unroll
                for (int g = 1; g <= MW_INLINE; ++g) good = good && (g > more || fits(x, g, s[g]));
            }
        }
        if (__all(good)) return true;
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

} // namespace pairs

// Greedy steps of the incremental-gain route, W workgroups per class (wgmap[b] = class, index among the class's workgroups,
// their count), at most max_steps of them.  Lists of more than `small` rows are left to the update launch, as
// rcd_k_inc_steps_mw leaves them (segments of the workgroups, one after the other).
template <typename S>
__global__ void __launch_bounds__(S::NT)
rcd_k_inc_steps_pairs(RcdClass *__restrict__ classes, RcdPlan *__restrict__ plans, const RcdWg *__restrict__ wgmap,
                       int max_steps, int small_bytes, unsigned epoch0, long long spin_ticks)
{
    using namespace pairs;
    constexpr int NW = S::NW, Q = S::Q, P = S::P;
    static_assert(NW == 8, "counts of two picks in 16 lanes, candidates of 32 rows in a wave");
    __shared__ __attribute__((aligned(16))) PairShared<S> sh;
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
    x.banks = mwbuf + MW_SLOT;
    x.abort_flag = &plans[0].bad;
    x.W = W;
    x.w = w;
    x.epoch = epoch0 + 1;
    x.deadline = tick0 + spin_ticks;
    bool alive = true;
    long long entries = 0, sweeps = 0;
    // everyone has read the descriptor before anyone may write it back
    if (W > 1) {
        __syncthreads();
        if (pl.wave == 0) {
            put(x, lane, 0, 1, 0, 0, 0);
            i32x4 s[4];
            const bool ok = get<GET_FIRST>(x, lane, s);
            if (lane == 0) sh.ok[0] = ok;
        }
        lds_barrier();
        alive = sh.ok[0] != 0;
    }
    auto write_held = [&]() {
        const RcdClass *c = rarely();
        if (w == 0) resident::write_outputs<S>(r, c->assign_out, c->order_out, c->out_index, pl);
    };
    while (alive) {
        const int j0 = resident::block_in_turn(r);
        if (j0 < 0 || !((r.valid >> j0) & 1u)) break;
        // the block that is next if j0's pick does not leave it the least again
        int j1 = resident::choose_block(r.f, (lane & 15) == j0 ? 0 : r.room);
        if (j1 >= 0 && (!((r.valid >> j1) & 1u) || r.t + 1 >= r.total || r.t + 1 - r.t0 >= r.max_steps)) j1 = -1;

        // ---- candidates of this slice
        {
            double t0[P], t1[P];
            resident::at_index<0, S::KM>(j0, [&](auto kc) {
#pragma unroll
                for (int i = 0; i < P; ++i) t0[i] = G[decltype(kc)::value][i];
            });
            if (j1 >= 0)
                resident::at_index<0, S::KM>(j1, [&](auto kc) {
#pragma unroll
                    for (int i = 0; i < P; ++i) t1[i] = G[decltype(kc)::value][i];
                });
            row_candidates<S>(t0, t1, j1 >= 0, pl, sh.slots);
        }
        // the coverage the picks' rows will be held against, on its way during the exchange
        f32x2 c[2][Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            c[0][q] = pl.at((gcf32)(cur_all + (size_t)j0 * ld), q);
            c[1][q] = pl.at((gcf32)(cur_all + (size_t)max(j1, 0) * ld), q);
        }
        lds_barrier();
        x.epoch += 1;
        if (pl.wave == 0) {
            const Slot a = sh.slots[0][lane & 31];
            const int mine = best_lane(lane < 32 ? a.hi : 0u, a.lo, a.v);
            i32x4 s[4];
            bool ok = true;
            const int hi = __builtin_amdgcn_readlane((int)a.hi, mine), lo = __builtin_amdgcn_readlane((int)a.lo, mine);
            const int v = __builtin_amdgcn_readlane(a.v, mine);
            if (W > 1) {
                put(x, lane, 0, 1, hi, lo, v);
                ok = get<GET_FIRST>(x, lane, s);
            } else {
                s[0] = lane == 0 ? (i32x4){hi, lo, v, 0} : (i32x4){0, 0, 0, 0};
            }
            // (lanes without a workgroup hold the key 0, below every number's)
            const int src = best_lane((unsigned)s[0].x, (unsigned)s[0].y, s[0].z);
            if (lane == src) sh.won[0] = Slot{(unsigned)s[0].x, (unsigned)s[0].y, s[0].z, 0};
            if (lane == 0) sh.ok[0] = ok;
        } else if (pl.wave == 1) {
            bool ok = true;
            if (j1 >= 0) {
                const Slot b = sh.slots[1 + (lane >> 5)][lane & 31];
                const int one = best_lane(b.hi, b.lo, b.v);
                const int two = best_lane(lane == one ? 0u : b.hi, b.lo, b.v);
                const i32x4 p1 = {__builtin_amdgcn_readlane((int)b.hi, one), __builtin_amdgcn_readlane((int)b.lo, one),
                                  __builtin_amdgcn_readlane(b.v, one), 0};
                const i32x4 p2 = {__builtin_amdgcn_readlane((int)b.hi, two), __builtin_amdgcn_readlane((int)b.lo, two),
                                  __builtin_amdgcn_readlane(b.v, two), 0};
                i32x4 s[4];
                if (W > 1) {
                    const i32x4 p = lane == 0 ? p1 : p2;
                    put(x, lane, 1, 2, p.x, p.y, p.z);
                    ok = get<GET_NEXT_TWO>(x, lane, s);
                } else {
                    s[0] = lane == 0 ? p1 : (i32x4){0, 0, 0, 0};
                    s[1] = lane == 0 ? p2 : (i32x4){0, 0, 0, 0};
                }
                const int src = best_lane((unsigned)s[0].x, (unsigned)s[0].y, s[0].z);
                if (lane == src) {
                    sh.won[1] = Slot{(unsigned)s[0].x, (unsigned)s[0].y, s[0].z, 0};
                    s[0] = s[1];
                }
                const int src2 = best_lane((unsigned)s[0].x, (unsigned)s[0].y, s[0].z);
                if (lane == src2) sh.won[2] = Slot{(unsigned)s[0].x, (unsigned)s[0].y, s[0].z, 0};
            }
            if (lane == 0) sh.ok[1] = ok;
        }
        lds_barrier();
        if ((sh.ok[0] & sh.ok[1]) == 0) { alive = false; break; }

        // ---- the picks (every wave of every workgroup alike)
        int pj[2] = {j0, j1}, pv[2] = {0, -1};
        f32x2 mp[2][Q];                          // their rows
        int B = 1;
        {
            const Slot a = sh.won[0], first = sh.won[1], second = sh.won[2];
            const Slot b = first.v == a.v ? second : first;
            const double best0 = inc_value(((unsigned long long)a.hi << 32) | a.lo);
            pv[0] = __builtin_amdgcn_readfirstlane(a.v);
            // no candidate left (cannot happen while t < total <= n; a test of values that are the same in every lane)
            if (__ballot(best0 > INC_LIVE_ABOVE) == 0ull || pv[0] >= n) { r.done = 1; break; }
            const gcf32 row = M + (size_t)pv[0] * ld;
#pragma unroll
            for (int q = 0; q < Q; ++q) mp[0][q] = pl.at(row, q);
            resident::take(r, j0, pv[0], best0, lane);
            resident::strike<S>(G, pv[0], pl.first, lane);
            const double best1 = inc_value(((unsigned long long)b.hi << 32) | b.lo);
            const int v1 = __builtin_amdgcn_readfirstlane(b.v);
            if (j1 >= 0 && r.next == j1 && __ballot(best1 > INC_LIVE_ABOVE) != 0ull && v1 < n) {
                B = 2;
                pv[1] = v1;
                const gcf32 row1 = M + (size_t)v1 * ld;
#pragma unroll
                for (int q = 0; q < Q; ++q) mp[1][q] = pl.at(row1, q);
                resident::take(r, j1, v1, best1, lane);
                resident::strike<S>(G, v1, pl.first, lane);
            }
        }

        // ---- coverage: the j of this slice with S(j, v*) > cur_k(j), ascending
        // f(position in the wave's part of the list, j, old, new) for every entry of pick u
        auto each_entry = [&](auto uc, auto &&f) {
            constexpr int u = decltype(uc)::value;
            int cnt = 0;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q < pl.nq) {
                    const bool ch0 = mp[u][q].x > c[u][q].x, ch1 = mp[u][q].y > c[u][q].y;
                    const unsigned long long b0 = __ballot(ch0), b1 = __ballot(ch1);
                    if ((b0 | b1) != 0ull) {
                        const int pos = cnt + __popcll(b0 & below) + __popcll(b1 & below);
                        const int v = (int)pl.v0 + 128 * q;
                        if (ch0) f(pos, v, c[u][q].x, mp[u][q].x);
                        if (ch1) f(pos + (ch0 ? 1 : 0), v + 1, c[u][q].y, mp[u][q].y);
                        cnt += __popcll(b0) + __popcll(b1);
                    }
                }
            return cnt;
        };
        auto stage_entries = [&](auto uc) {
            constexpr int u = decltype(uc)::value;
            Entry *held = sh.stage[u * NW + pl.wave];
            const int cnt = each_entry(uc, [&](int pos, int j, float o, float nw) {
                if (pos < MW_INLINE) held[pos] = Entry{j, o, nw, 0};
            });
            if (lane == 0) sh.count[u * NW + pl.wave] = cnt;
        };
        stage_entries(std::integral_constant<int, 0>{});
        if (B == 2) stage_entries(std::integral_constant<int, 1>{});
        else if (lane == 0) sh.count[NW + pl.wave] = 0;
        lds_barrier();

        // ---- the lists: lane u NW + i holds the length of wave i's part for pick u
        const int found = lane < 2 * NW ? sh.count[lane] : 0;
        const int incl = wave_prefix(found, lane);
        const int len0 = __builtin_amdgcn_readlane(incl, NW - 1), both = __builtin_amdgcn_readlane(incl, 2 * NW - 1);
        const int len1 = both - len0;
        // this wave's place in the segments
        const int base0 = __builtin_amdgcn_readlane(incl - found, pl.wave);
        const int base1 = __builtin_amdgcn_readlane(incl - found, NW + pl.wave) - len0;
        auto write_segment = [&](auto uc, int base) {
            const size_t at = (size_t)pj[decltype(uc)::value] * ld + s0 + base;
            const RcdClass *c = rarely();
            const gi32 dlist = (gi32)inc_dlist(*c);
            const gf32 dold = (gf32)inc_dold(*c), dnew = (gf32)inc_dnew(*c);
            each_entry(uc, [&](int pos, int j, float o, float nw) {
                dev_store(dlist + at + pos, j);
                dev_store(dold + at + pos, o);
                dev_store(dnew + at + pos, nw);
            });
        };
        const bool in_memory = both > MW_INLINE;    // too many entries for the post
        if (in_memory) {
            write_segment(std::integral_constant<int, 0>{}, base0);
            if (B == 2) write_segment(std::integral_constant<int, 1>{}, base1);
            wait_for_my_stores();
            lds_barrier();
        }
        x.epoch += 1;
        if (pl.wave == 0) {
            if (!in_memory && found > 0)
                for (int g = 0; g < found; ++g) sh.mine[incl - found + g] = sh.stage[lane][g];
            __builtin_amdgcn_wave_barrier();
            int a = len0, b = len1, d = 0;
            if (lane > 0 && lane <= MW_INLINE) {
                const Entry e = sh.mine[lane - 1];
                a = e.j;
                b = __float_as_int(e.o);
                d = __float_as_int(e.n);
            }
            i32x4 s[4];
            bool ok = true;
            if (W > 1) {
                put(x, lane, 0, in_memory ? 1 : 1 + both, a, b, d);
                ok = get<GET_LIST>(x, lane, s);
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    s[g] = lane == 0 ? (i32x4){__builtin_amdgcn_readlane(a, g), __builtin_amdgcn_readlane(b, g),
                                               __builtin_amdgcn_readlane(d, g), 0}
                                     : (i32x4){0, 0, 0, 0};
            }
            // (posts that have not come say nothing: no place in the lists may be taken from their words)
            const int l0 = ok && lane < W ? s[0].x : 0, l1 = ok && lane < W ? s[0].y : 0;
            const int i0 = wave_prefix(l0, lane), i1 = wave_prefix(l1, lane);
            const int nd0 = __builtin_amdgcn_readlane(i0, 63), nd1 = __builtin_amdgcn_readlane(i1, 63);
            const int keep0 = nd0 > small ? 0 : nd0, keep1 = nd1 > small ? 0 : nd1;
            // list 0 from entry 0 on, list 1 behind what of list 0 is applied here
            const int at0 = i0 - l0, at1 = keep0 + i1 - l1;
            if (lane < W) {
                sh.len[0][lane] = keep0 > 0 ? l0 : 0;
                sh.len[1][lane] = keep1 > 0 ? l1 : 0;
                sh.pre[0][lane] = at0;
                sh.pre[1][lane] = at1;
                sh.fetch[lane] = l0 + l1 > MW_INLINE;
                if (l0 + l1 <= MW_INLINE) {
#pragma unroll
                    for (int g = 0; g < MW_INLINE; ++g) {
                        const Entry e = {s[g + 1].x, __int_as_float(s[g + 1].y), __int_as_float(s[g + 1].z), 0};
                        if (g < l0 ? keep0 > 0 : g < l0 + l1 && keep1 > 0) sh.list[g < l0 ? at0 + g : at1 + g - l0] = e;
                    }
                }
            }
            const unsigned long long lng = __ballot(l0 + l1 > MW_INLINE && (l0 > 0 && keep0 > 0 || l1 > 0 && keep1 > 0));
            if (lane == 0) { sh.nd[0] = nd0; sh.nd[1] = nd1; sh.any_long = lng != 0ull; sh.ok[0] = ok; }
        }
        lds_barrier();
        if (sh.ok[0] == 0) { alive = false; break; }
        const int nd0 = __builtin_amdgcn_readfirstlane(sh.nd[0]), nd1 = __builtin_amdgcn_readfirstlane(sh.nd[1]);
        const bool pend0 = nd0 > small, pend1 = nd1 > small;
        const int n0 = pend0 ? 0 : nd0, total = n0 + (pend1 ? 0 : nd1);
        entries += nd0 + nd1;
        if (sh.any_long) {
            // segments that did not travel in the posts: a wave per segment
            const RcdClass *c = rarely();
            const gi32 dlist = (gi32)inc_dlist(*c);
            const gf32 dold = (gf32)inc_dold(*c), dnew = (gf32)inc_dnew(*c);
            for (int i = pl.wave; i < W; i += NW) {
                const int a = sh.len[0][i], b = sh.len[1][i];
                if (sh.fetch[i] == 0 || a + b == 0) continue;
                const int pa = sh.pre[0][i], pb = sh.pre[1][i];
                const size_t at0 = (size_t)pj[0] * ld + (size_t)i * mwseg, at1 = (size_t)max(pj[1], 0) * ld + (size_t)i * mwseg;
                for (int e = lane; e < a + b; e += 64) {
                    const size_t at = e < a ? at0 + e : at1 + (e - a);
                    sh.list[e < a ? pa + e : pb + (e - a)] = Entry{dev_load(dlist + at), dev_load(dold + at), dev_load(dnew + at), 0};
                }
            }
            lds_barrier();
        }

        // ---- gains: the lists' terms, both lists end to end, added up per pick in list order, then onto the block's gains
        {
            double acc[P];
#pragma unroll
            for (int i = 0; i < P; ++i) acc[i] = 0.0;
            auto flush = [&](int k) {
                resident::update_at_index<0, S::KM>(k, [&](auto kc) {
#pragma unroll
                    for (int i = 0; i < P; ++i) G[decltype(kc)::value][i] += acc[i];
                });
            };
            constexpr int U = S::ROWS;           // rows in flight
            for (int first = 0; first < total; first += 64) {
                const Entry en = sh.list[min(first + lane, total - 1)];
                const int here = min(64, total - first);
                const unsigned long long own0 = __ballot(first + lane < n0 && en.j == pv[0]);
                const unsigned long long own1 = __ballot(first + lane >= n0 && en.j == pv[1]);
                f32x2 m[U][Q];
                auto fetch = [&](int i, int e) __attribute__((always_inline)) {
                    const gcf32 row = M + (size_t)__builtin_amdgcn_readlane(en.j, e) * ld;
#pragma unroll
                    for (int q = 0; q < Q; ++q) m[i][q] = pl.at(row, q);
                };
                // (the boundary between the lists is looked at entry by entry: as a place of its own behind the loops the
                // update of the gains took fewer instructions and more registers than there are)
                auto use = [&](int i, int e) __attribute__((always_inline)) {
                    if (first + e == n0 && n0 > 0) {
                        flush(pj[0]);
#pragma unroll
                        for (int a = 0; a < P; ++a) acc[a] = 0.0;
                    }
                    const float cn = inc_lane_value(en.n, e), co = inc_lane_value(en.o, e);
#pragma unroll
                    for (int q = 0; q < Q; ++q) {
                        acc[2 * q] += inc_term(m[i][q].x, cn, co);
                        acc[2 * q + 1] += inc_term(m[i][q].y, cn, co);
                    }
                };
                int e0 = 0;
                if (here >= 2 * U) {
                    // a long list: U rows in flight all the time, no condition between the loads
#pragma unroll
                    for (int i = 0; i < U; ++i) fetch(i, i);
                    for (; e0 + 2 * U <= here; e0 += U)
#pragma unroll
                        for (int i = 0; i < U; ++i) {
                            use(i, e0 + i);
                            fetch(i, e0 + U + i);
                        }
#pragma unroll
                    for (int i = 0; i < U; ++i) use(i, e0 + i);
                    e0 += U;
                }
                for (; e0 < here; e0 += U) {
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        if (e0 + i < here) {
                            // (v* is on its own list, unless an equal sample is in the block already)
                            if ((own0 >> (e0 + i)) & 1ull) {
#pragma unroll
                                for (int q = 0; q < Q; ++q) m[i][q] = mp[0][q];
                            } else if ((own1 >> (e0 + i)) & 1ull) {
#pragma unroll
                                for (int q = 0; q < Q; ++q) m[i][q] = mp[1][q];
                            } else {
                                fetch(i, e0 + i);
                            }
                        }
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        if (e0 + i < here) use(i, e0 + i);
                }
            }
            if (total > 0) flush(total > n0 ? pj[1] : pj[0]);
        }

        // ---- the new coverage of this slice, and what is left to the update launch
        auto leave = [&](auto uc, int base, int mine, int nd) {
            constexpr int u = decltype(uc)::value;
            if (!in_memory) write_segment(uc, base);
            r.valid &= ~(1u << pj[u]);
            sweeps += 1;
            if (threadIdx.x == 0) {
                mwbuf[MW_PEND + pj[u] * RCD_SLICES_MAX + w] = mine;
                if (w == 0) st.dcount[pj[u]] = nd;
            }
        };
        auto cover = [&](auto uc) {
            constexpr int u = decltype(uc)::value;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q < pl.nq && (mp[u][q].x > c[u][q].x || mp[u][q].y > c[u][q].y)) {
                    const f32x2 top = {fmaxf(mp[u][q].x, c[u][q].x), fmaxf(mp[u][q].y, c[u][q].y)};
                    *off<f32x2>(cur_all + (size_t)pj[u] * ld, (pl.v0 + 128u * q) * 4u) = top;
                }
        };
        cover(std::integral_constant<int, 0>{});
        if (pend0) leave(std::integral_constant<int, 0>{}, base0, len0, nd0);
        if (B == 2) {
            cover(std::integral_constant<int, 1>{});
            if (pend1) leave(std::integral_constant<int, 1>{}, base1, len1, nd1);
        }
        if (r.held > 60) {
            write_held();
            r.held = 0;
        }
    }
    if (!alive) return;          // a bounded wait ran out: plans[0].bad says so, nothing is written back
    write_held();
    if (!r.done) resident::store_gains<S>(G, inc_gains(st), K, ld, pl);
    if (w != 0) return;
    resident::store_run(r, st, plans, entries * n, sweeps, true, wall_clock64() - tick0);
    const unsigned waiting = (unsigned)__ballot(lane < K && r.room > 0 && !((r.valid >> (lane & 15)) & 1u)) & 0xFFFFu;
    if (threadIdx.x == 0 && !r.done) {
        int nneed = 0;
        for (unsigned k = waiting; k; k &= k - 1u) st.need[nneed++] = (int)__builtin_ctz(k);
        st.nneed = nneed;
    }
}

namespace sliced {

struct Choice {
    void (*inc)(RcdClass *, RcdPlan *, const RcdWg *, int, int, unsigned, long long);
    int threads;
    bool several;            // up to eight picks to a trip, not two
};
template <int Q, int KM, int ROWS> Choice choice() { return Choice{rcd_k_inc_steps_sliced<SliceShape<Q, KM, ROWS>>, 512, true}; }

// Slices over 1024 with up to eight blocks, two picks to a trip (no register spilled) / up to eight, mixtures, in ms: forty classes of
// 12 000, eight blocks 222 / 214, 20 of 15 000, five 182 / 172, 16 of 20 000, eight 291 / 280, 60 of 6000, four 71 / 68, forty of 8000, one
// 78 / 66; every sample with a near copy 230 / 235, 183 / 193, 301 / 288, 76 / 85, 83 / 90; four picks to a trip, with which <2, 8> spills 16
// registers, 223, 179, 289, 70, 68.5 on mixtures.
// The smallest variant whose registers hold a slice's gains for K blocks.  At most RCD_MW_MAX slices to a class for the last.
inline Choice choose(int slice, int K)
{
    if (slice <= 1024) return K <= 4 ? choice<1, 4, 8>() : K <= 8 ? choice<1, 8, 8>() : choice<1, 16, 8>();
    if (slice <= 2048) return K <= 4 ? choice<2, 4, 4>() : K <= 8 ? choice<2, 8, 4>() : Choice{rcd_k_inc_steps_pairs<pairs::PairShape<2, 16, 6>>, 512, false};
    return Choice{nullptr, 0, false};
}

} // namespace sliced
