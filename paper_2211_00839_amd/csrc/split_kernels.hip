// Class split of Algorithm 1 ("Split the ground set V into V_1..V_L according to
// class labels"): a stable counting sort of sample indices by label, so that
// inside every class the samples keep the caller's order.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "rcd_state.h"

namespace split {

constexpr int CHUNK = 1024;   // samples per chunk, one wave per chunk

// chunk_hist[chunk][l] = number of samples with label l in the chunk.  A bad label anywhere in the chunk is told by the
// sign of its first count (the complement of it): no flag has to be cleared beforehand.
// allow_unassigned: a label of -1 is not an error, the sample just belongs nowhere (worker shards of a
// partition that left samples over).
// Bound by the trip to memory, hence all of a wave's labels are asked for before the first is counted; up to 16 labels are
// counted by ballots, since 64 lanes adding to eight counters in LDS take their turns.
__global__ void __launch_bounds__(64)
k_hist(const int32_t *__restrict__ labels, long long N, int L, int32_t *__restrict__ chunk_hist, int allow_unassigned)
{
    extern __shared__ int s_cnt[];
    const int lane = threadIdx.x;
    const long long base = (long long)blockIdx.x * CHUNK;
    constexpr int GROUPS = CHUNK / 64;
    int lab[GROUPS];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const long long i = base + g * 64 + lane;
        lab[g] = i < N ? labels[i] : -2;
    }
    bool bad = false;
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
        bad |= base + g * 64 + lane < N && (lab[g] < 0 || lab[g] >= L) && !(allow_unassigned && lab[g] == -1);
    const bool any_bad = __any(bad);
    int32_t *out = chunk_hist + (size_t)blockIdx.x * L;
    if (L <= 16) {
        int mine = 0;
        for (int l = 0; l < L; ++l) {
            int c = 0;
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) c += __popcll(__ballot(lab[g] == l));
            mine = lane == l ? c : mine;
        }
        if (lane < L) out[lane] = lane == 0 && any_bad ? ~mine : mine;
        return;
    }
    for (int l = lane; l < L; l += 64) s_cnt[l] = 0;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
        if (lab[g] >= 0 && lab[g] < L) atomicAdd(&s_cnt[lab[g]], 1);
    __syncthreads();
    for (int l = lane; l < L; l += 64) out[l] = l == 0 && any_bad ? ~s_cnt[l] : s_cnt[l];
}

// Per class: exclusive prefix of chunk_hist over chunks (in place) and the class total.  One workgroup per class, a run
// of consecutive chunks per thread: with one thread per class walking all its chunks, a million labels in eight classes
// took 128 us, 977 dependent trips to memory; here the chunks are read side by side (4.6 us).
// Class 0's workgroup, which sees the signs, says whether a label was bad.  host (pinned memory): the class totals and behind
// them that flag, written from here: a copy between this launch and the next cost a million labels ten of 43 us.
__global__ void __launch_bounds__(256)
k_scan(int32_t *__restrict__ chunk_hist, int nchunks, int L, int32_t *__restrict__ class_count, RcdPlan *__restrict__ plan,
       int32_t *__restrict__ host)
{
    __shared__ int s_wave[4];
    const int l = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (nchunks + 255) / 256;
    const int c0 = min(tid * per, nchunks), c1 = min(c0 + per, nchunks);
    int sum = 0;
    bool bad = false;
    for (int c = c0; c < c1; ++c) {
        const int v = chunk_hist[(size_t)c * L + l];
        bad |= v < 0;
        sum += v < 0 ? ~v : v;
    }
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        if (lane >= off) incl += up;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int run = incl - sum;
    for (int w = 0; w < wave; ++w) run += s_wave[w];
    for (int c = c0; c < c1; ++c) {
        const int v = chunk_hist[(size_t)c * L + l];
        chunk_hist[(size_t)c * L + l] = run;
        run += v < 0 ? ~v : v;
    }
    if (tid == 255) {
        class_count[l] = run;
        host[l] = run;
    }
    const int any_bad = __syncthreads_or(bad);
    if (l == 0 && tid == 0) {
        plan->bad = any_bad;
        host[L] = any_bad;
    }
}

// idx[offset of class l + rank] = i, rank = number of earlier samples with label l, the classes end to end in order.
// One wave per chunk; every lane finds the lanes of its group of 64 that share its label with one ballot per bit of a
// label (label_bits of them), so a group costs the same however many labels it holds (a loop over the distinct labels with
// two barriers in each took 25 us for a million labels of eight classes, this takes 8.0), and all labels of the chunk are
// on their way at once.  A bad label anywhere (plan->bad, from k_scan) and nothing is written: the host reads that flag
// only behind this launch.
__global__ void __launch_bounds__(64)
k_scatter(const int32_t *__restrict__ labels, long long N, int L, int label_bits, const int32_t *__restrict__ chunk_base,
          const int32_t *__restrict__ class_count, const RcdPlan *__restrict__ plan, int32_t *__restrict__ idx)
{
    extern __shared__ int s_cnt[];
    const int bad = plan->bad;     // (looked at below, when it has come with the labels)
    const int lane = threadIdx.x;
    const long long base = (long long)blockIdx.x * CHUNK;
    constexpr int GROUPS = CHUNK / 64;
    int lab[GROUPS];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const long long i = base + g * 64 + lane;
        lab[g] = i < N ? labels[i] : -1;
    }
    // where this chunk's first sample of each class goes
    int before = 0;
    for (int l0 = 0; l0 < L; l0 += 64) {
        const int l = l0 + lane;
        const int c = l < L ? class_count[l] : 0;
        int incl = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
        }
        if (l < L) s_cnt[l] = before + incl - c + chunk_base[(size_t)blockIdx.x * L + l];
        before += __shfl(incl, 63);
    }
    if (bad) return;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const int l = lab[g];
        const bool has = l >= 0 && l < L;
        unsigned long long same = __ballot(has);
        for (int b = 0; b < label_bits; ++b) {
            const unsigned long long ones = __ballot((l >> b) & 1);
            same &= ((l >> b) & 1) ? ones : ~ones;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        int start = 0;
        if (has) {
            start = s_cnt[l];
            idx[start + rank] = (int32_t)(base + g * 64 + lane);
        }
        __syncthreads();           // every lane has read the counters (one wave: no wait, the order of the LDS accesses)
        if (has && rank == 0) s_cnt[l] = start + __popcll(same);
        __syncthreads();
    }
}

// bits that tell the labels 0 .. L-1 apart
inline int bits_of(int L)
{
    int b = 0;
    while ((1ll << b) < L) ++b;
    return b;
}

} // namespace split
