// Target-only speculative sampling: one token per tree node drawn from the target model's own
// distribution (temperature, top-k, top-p), so that acceptance needs no draft probabilities.
//
// Beyond greedy decoding the paper runs SSSD with a reduced form of speculative sampling that keeps
// the target distribution exact and needs no probabilities from the draft side (Sec. 4.4, at
// temperature 0.6 / top-p 0.95; Fig. 5 uses temperature 0.7, top-p 0.8, top-k 20).
// n-gram drafts carry no probabilities: the draft distribution of a proposed token is a point mass,
// for which the acceptance test of speculative sampling (accept with probability min(1, p/q), else
// resample from the normalised residual) is the same as drawing ONE token t from the target
// distribution p of the node and accepting the child that carries t, if any; otherwise t itself is
// emitted and the walk stops.  Every emitted token is an exact sample of p given its prefix.
//
// Distribution of a row (logits z, temperature T > 0, top_k, top_p):
//   order O: by logit descending, token id ascending among equal logits
//   S_k = the first top_k tokens of O (all tokens if top_k is 0 or >= vocab)
//   w_i = exp((z_i - max z) / T);  Z_k = sum of w over S_k
//   S   = the shortest prefix of O (at least one token) whose w-sum reaches top_p * Z_k
//   the sample: r = u * Z_S, the first token of S in ascending TOKEN ID order whose running
//   w-sum exceeds r (u is the caller's uniform number in [0, 1) for this row).
//
// One workgroup of 1024 threads per row.  Both selections are radix selects over the 32-bit logit
// pattern (four 8-bit digits, most significant first): top-k on counts, top-p on masses.  Masses
// are 1.31 fixed-point integers accumulated in 64 bits with integer LDS atomics, so every sum is exact and
// independent of the order of accumulation: the kernel is deterministic, and a tie at a threshold
// is resolved by token id exactly as the definition says.  The row stays in L2 across the passes.
#include "kernels.h"

namespace {

constexpr int ST = 1024;   // threads per row
constexpr int MAX_BATCH = 64;   // batches of 512 ids per wave: vocabularies up to 16 * 64 * 512 tokens

// Order-preserving map of a finite float to uint32: larger float -> larger key.
__device__ __forceinline__ uint32_t order_key(float z)
{
    const uint32_t u = f32_bits(z);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

struct RowCtx {
    const float *z;
    int V;
    float mx, scale;   // w = exp2((z - mx) * scale)
};

// Weight of a token as a 1.31 fixed-point integer: w * 2^31 is exact in fp32 (a power-of-two scale)
// and fits 32 bits because w <= 1.
__device__ __forceinline__ uint64_t fix_mass(const RowCtx &r, float z)
{
    const float w = __builtin_amdgcn_exp2f((z - r.mx) * r.scale);   // in [0, 1]
    return (uint64_t)(uint32_t)(w * 2147483648.0f);
}

// Wave 0 scans 256 bins from the top: the bin g with above + (sum of higher bins) < target <= that + bins[g]
// (bin 0 if the target is never reached).  Every lane returns g and the sum of the bins above g;
// lane l owns bins 4l .. 4l+3.
template <typename T> __device__ int pick_bin(const T *bins, T target, T above, T &higher, int lane)
{
    T v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = bins[4 * lane + e];
    const T mine = v[0] + v[1] + v[2] + v[3];
    T suffix = mine;   // sum over lanes >= lane
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const T o = __shfl_down(suffix, off);
        if (lane + off < 64) suffix += o;
    }
    T hi = suffix - mine;   // sum of the bins of higher lanes
    int g = -1;
    T hg = 0;
#pragma unroll
    for (int e = 3; e >= 0; --e) {
        if (g < 0 && above + hi + v[e] >= target) { g = 4 * lane + e; hg = hi; }
        hi += v[e];
    }
    // the highest bin that qualifies wins
    const unsigned long long found = __ballot(g >= 0);
    const int src = found ? 63 - __clzll(found) : 0;
    int gs = __shfl(g, src);
    T hs = __shfl(hg, src);
    if (!found) { gs = 0; hs = __shfl(suffix, 0) - __shfl(v[0], 0); }
    higher = hs;
    return gs;
}

// Histogram accumulation through a private run per thread: consecutive elements that fall into the
// same bin (the leading digits of a row's logits mostly do) are summed in registers and reach LDS as
// one atomic add when the bin changes, so a hot bin is not hit by an atomic per element.
struct BinRun {
    uint32_t bin, count;
    uint64_t mass;
    bool open;
};
__device__ __forceinline__ void run_flush(BinRun &r, uint32_t *chist, uint64_t *mhist)
{
    if (!r.open) return;
    if (chist) atomicAdd(&chist[r.bin], r.count);
    if (mhist) atomicAdd((unsigned long long *)&mhist[r.bin], (unsigned long long)r.mass);
    r.open = false;
}
__device__ __forceinline__ void run_add(BinRun &r, uint32_t bin, uint64_t mass, uint32_t *chist, uint64_t *mhist)
{
    if (r.open && r.bin == bin) {
        r.count += 1;
        r.mass += mass;
        return;
    }
    run_flush(r, chist, mhist);
    r.bin = bin;
    r.count = 1;
    r.mass = mass;
    r.open = true;
}

// body(i, z, valid) for i = begin + first, begin + first + stride, ... below end, in ascending order.
// The loads go out eight at a time: a pass is bound by load latency, not by bandwidth (the row is in L2).
// Every thread makes the same number of calls (valid = false past the end), so body may use wave-wide
// operations.
constexpr int SU = 8;
template <typename F>
__device__ __forceinline__ void for_row(const float *z, int begin, int end, int first, int stride, F body)
{
    for (int base = begin; base < end; base += stride * SU) {
        float zz[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int i = base + u * stride + first;
            zz[u] = i < end ? z[i] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int i = base + u * stride + first;
            body(i, zz[u], i < end);
        }
    }
}

// The whole row, any order: 16-byte loads (four tokens per thread and load) when the row allows it.  `more` (wave-uniform)
// is asked before every round of loads and ends the walk.  BACK: the last round first; a pass after a forward one then starts with what
// the die's L2 still holds, which has no room for the rows of all its compute units (160 rows of 128256, top-k 20 + top-p 0.8
// 35.2 -> 34.1 us, 128 rows, top-k 50 40.0 -> 37.8, 96 rows, top-p 0.95 50.7 -> 49.4).
template <bool BACK, typename F, typename P> __device__ __forceinline__ void for_whole_row(const float *z, int V, bool vec4, int tid, F body, P more)
{
    if (!vec4) {
        for (int base = 0; base < V && more(); base += ST * SU) for_row(z, base, min(V, base + ST * SU), tid, ST, body);
        return;
    }
    const f32x4 *z4 = reinterpret_cast<const f32x4 *>(z);
    const int V4 = V >> 2;
    constexpr int STEP = ST * SU;
    for (int base = BACK ? (V4 - 1) / STEP * STEP : 0; (BACK ? base >= 0 : base < V4) && more(); base += BACK ? -STEP : STEP) {
        f32x4 zz[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int i = base + u * ST + tid;
            zz[u] = i < V4 ? z4[i] : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int i = base + u * ST + tid;
#pragma unroll
            for (int e = 0; e < 4; ++e) body(4 * i + e, zz[u][e], i < V4);
        }
    }
}
template <bool BACK = false, typename F> __device__ __forceinline__ void for_whole_row(const float *z, int V, bool vec4, int tid, F body)
{
    for_whole_row<BACK>(z, V, vec4, tid, body, [] { return true; });
}

// ---- several workgroups per row ----
// One compute unit pulls a 513 KB row out of L2 in 10-15 us, and the exact selections need seven to
// twelve passes: with few rows (a step of B = 1 has k+1 of them) the kernel's time is that of one row on
// one compute unit.  So a row is given to a CLUSTER of C workgroups, each on its own contiguous range of
// token ids; what a pass finds (maximum, histogram bins, tie counts, member mass) is merged through a
// small scratch block in global memory and a barrier among the C workgroups, after which every workgroup
// takes the same decision from the same merged numbers.  All merged quantities are integers (or a
// maximum), so the result does not depend on C: the cluster of one is the plain kernel.
//
// The barrier is a counter per cluster that only grows: barrier number n of a launch waits for n*C
// arrivals.  Shared words are written with device-scope atomics (or device-scope stores, waited for,
// before the workgroup is counted in) and read with device-scope loads, as in the split-K hand-over of
// the GEMM kernels.  Waiting is bounded: a cluster whose workgroups are not all resident (the launch
// assumes the device to itself: grid <= compute units) gives up after SPIN_LIMIT polls, raises *err and
// leaves its rows unsampled (-1) instead of hanging.
constexpr int MAX_CLUSTER = 16;
constexpr int HIST_PASSES = 8;            // four count passes (top-k) and four mass passes (top-p)
constexpr unsigned SPIN_LIMIT = 1u << 20;
constexpr int FINE_BINS = 512;            // short path: bins of 1/16 octave of weight, 31 octaves (496) and a spare
constexpr int FINE_COPIES = 8;            // copies of the bins in LDS, by lane, against same-address adds within a wave
constexpr int LIST_MAX = 4096;            // short path: candidates kept (of the nucleus' last bin)
constexpr int LIST_K_MAX = 1024;          // ... of a top-k selection, one per thread
constexpr int SHORT_K_MAX = 256;          // largest top_k that the short path takes
constexpr int MAX_SUB = 16 * MAX_BATCH;   // (workgroup, wave, batch) sums of a row
struct SampleScratch {                    // one per cluster; the two counters are zero when a launch starts
    uint32_t arrivals;
    uint32_t departures;                  // the last workgroup to leave puts both counters back to zero
    uint32_t pad[14];
    float gmax[MAX_CLUSTER];
    uint32_t gties[MAX_CLUSTER];
    uint64_t gsub[MAX_CLUSTER];
    uint32_t chist[HIST_PASSES][256];
    uint64_t mhist[HIST_PASSES][256];
    // short path
    uint64_t fine[FINE_BINS];             // cleared when the row begins
    uint32_t kmax[MAX_CLUSTER], kmin[MAX_CLUSTER], bound_k[MAX_CLUSTER], bound_1[MAX_CLUSTER], count[MAX_CLUSTER];
    uint64_t mass[MAX_CLUSTER];
    uint64_t sub[MAX_SUB];
    uint32_t keys[LIST_MAX], ids[LIST_MAX];   // workgroup c of C: LIST_MAX / C entries from c * LIST_MAX / C on
};

struct Cluster {
    SampleScratch *s;
    int C, c;
    uint32_t passed;   // barriers passed so far in this launch (same in every workgroup of the cluster)
    bool failed;
};

// All threads of all workgroups of the cluster.  Returns false when the wait ran out.
__device__ __forceinline__ bool cluster_sync(Cluster &cl, int32_t *err)
{
    if (cl.C == 1) return true;
    __shared__ int ok_s;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    cl.passed += 1;
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(&cl.s->arrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t want = cl.passed * (uint32_t)cl.C;
        unsigned spins = 0;
        while (__hip_atomic_load(&cl.s->arrivals, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want && spins < SPIN_LIMIT) {
            __builtin_amdgcn_s_sleep(2);
            ++spins;
        }
        ok_s = spins < SPIN_LIMIT;
        if (!ok_s && err) atomicOr(err, 2);
    }
    __syncthreads();
    const bool ok = ok_s != 0;
    __syncthreads();
    if (!ok) cl.failed = true;
    return ok;
}

// Local 256-bin histograms -> the cluster's bins of this pass -> back into LDS (every workgroup then holds
// the merged bins).  Whole workgroup; tid < 256 owns bin tid.
__device__ __forceinline__ bool merge_bins(Cluster &cl, int pass, uint32_t *chist, uint64_t *mhist, bool counts, bool masses, int tid,
                                           int32_t *err)
{
    if (cl.C == 1) return true;
    if (tid < 256) {
        if (counts && chist[tid]) __hip_atomic_fetch_add(&cl.s->chist[pass][tid], chist[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (masses && mhist[tid])
            __hip_atomic_fetch_add((unsigned long long *)&cl.s->mhist[pass][tid], (unsigned long long)mhist[tid], __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!cluster_sync(cl, err)) return false;
    if (tid < 256) {
        if (counts) chist[tid] = __hip_atomic_load(&cl.s->chist[pass][tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (masses)
            mhist[tid] = __hip_atomic_load((unsigned long long *)&cl.s->mhist[pass][tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return true;
}

// ---- the short path ----
// The selections above read the row once per 8-bit digit (four times for top-k, four for top-p, besides the maximum, the
// members' sums and the ties): ten or more passes of 5-15 us on a 513 KB row, which is all the kernel's time.  Nearly
// always a short list decides the row instead, and two or three passes do:
//   top-k   the top_k-th largest of the maxima of disjoint groups of tokens is a lower bound of the top_k-th largest
//           logit, so pass 1 (maxima per thread) gives a bound and pass 2 collects the few tokens at or above it, all
//           ties included.  Everything after that works on the list: rank in order O, nucleus, draw.
//   top-p   pass 2 adds the masses into bins of 1/16 octave of the weight (a bin is a contiguous range of logits, as the
//           bin number is monotonic in the logit), which gives Z and the bin that holds the nucleus' last token; pass 3
//           sums the tokens above that bin per batch of 512 ids and collects the tokens inside it, whose radix select runs
//           in LDS.
//   neither  passes 1 and 3, every token counting as above the bin.
// Masses, targets and ties are those of the general path, integer for integer, so the token is the same one.  Rows whose
// list would overflow (very many equal or nearly equal logits), rows with an infinite or NaN maximum and temperatures whose
// reciprocal overflows go to the general path, with what is known by then (Known): the maximum, and the digits that all
// keys in question share, which need no pass.  They are told early, since a pass more is what it would cost them: by the
// range of the logits (pass 1), by the mass of the last bin (pass 2), or when the top-k list is full.  top_k above
// SHORT_K_MAX is a kernel of its own, without the lists' registers.
// Measured at vocabulary 128256, us, without lists -> with: 160 rows top-k 20 + top-p 0.8 212 -> 34, top-p 0.9 on N(0, 2)
// 192 -> 77, neither 65 -> 46; 9 rows top-p 0.95 46 -> 30, neither 24 -> 16.  On the general path, 160 rows: top-p 0.9 on
// equal logits 224 -> 216, on N(0, 0.1) 186 -> 188, on logits rounded to quarters 245 -> 218, top-k 50 on equal logits
// 164 -> 102, top-k 300 167 -> 159.
struct ShortLds {
    uint64_t fine[FINE_COPIES][FINE_BINS];
    uint32_t keys[LIST_MAX], ids[LIST_MAX];
    uint64_t sub[MAX_SUB];
    uint64_t bins[256];
    uint32_t gmax[ST];
    uint64_t red[16];
    uint64_t above, equal;
    uint32_t n, prefix, bound, bound1;
    int bin;
};

// The leading 8-bit digits that two keys share, at most three: into prefix; returns the first digit (3 .. 0) below them.
__device__ __forceinline__ int common_digits(uint32_t a, uint32_t b, uint32_t &prefix)
{
    const uint32_t diff = a ^ b;
    const int d = diff >> 24 ? 3 : diff >> 16 ? 2 : diff >> 8 ? 1 : 0;
    prefix = d == 3 ? 0u : a >> (8 * (d + 1));
    return d;
}

__device__ __forceinline__ float key_logit(uint32_t key) { return bits_f32((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key); }

template <typename T> __device__ __forceinline__ T dev_load(T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T> __device__ __forceinline__ void dev_store(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ __forceinline__ uint64_t wave_sum(uint64_t v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Appends (key, id) of the lanes that `take` to the workgroup's list (whole wave; order is immaterial).
__device__ __forceinline__ void list_push(ShortLds &L, bool take, uint32_t key, int id, int lane)
{
    const uint64_t bal = __ballot(take);
    if (!bal) return;
    const int first = __ffsll((long long)bal) - 1;
    uint32_t base = 0;
    if (lane == first) base = atomicAdd(&L.n, (uint32_t)__popcll(bal));
    base = __shfl(base, first) + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
    if (take && base < (uint32_t)LIST_MAX) { L.keys[base] = key; L.ids[base] = (uint32_t)id; }
}

// With C > 1: this workgroup's list to its place in the scratch, before the barrier ...
__device__ __forceinline__ void list_publish(ShortLds &L, const Cluster &cl, int tid)
{
    if (cl.C == 1) return;
    __syncthreads();
    const uint32_t cap = LIST_MAX / cl.C, n = L.n;
    if (tid == 0) dev_store(&cl.s->count[cl.c], n);
    if (n <= cap)
        for (uint32_t i = tid; i < n; i += ST) {
            dev_store(&cl.s->keys[cl.c * cap + i], L.keys[i]);
            dev_store(&cl.s->ids[cl.c * cap + i], L.ids[i]);
        }
}

// ... and the whole cluster's list into the first workgroup's LDS, behind it.  False when a workgroup's part or the whole
// (more than `most`) overflowed: the same answer in every workgroup.
__device__ __forceinline__ bool list_gather(ShortLds &L, const Cluster &cl, uint32_t most, int tid)
{
    if (cl.C == 1) return L.n <= most;
    const uint32_t cap = LIST_MAX / cl.C;
    uint32_t at[MAX_CLUSTER], n = 0;
    bool fits = true;
    const int lane = tid & 63;
    const uint32_t mine = lane < cl.C ? dev_load(&cl.s->count[lane]) : 0;
#pragma unroll
    for (int c = 0; c < MAX_CLUSTER; ++c) {
        at[c] = n;
        const uint32_t k = __shfl(mine, c);
        fits = fits && k <= cap;
        n += k;
    }
    if (!fits || n > most) return false;
    if (cl.c == 0) {
        __syncthreads();   // the workgroup's own list was published out of the same words
        for (int c = tid >> 6; c < cl.C; c += ST / 64) {   // a wave per part
            uint32_t from = 0;
#pragma unroll
            for (int x = 0; x < MAX_CLUSTER; ++x) from = x == c ? at[x] : from;
            const uint32_t k = __shfl(mine, c);
            for (uint32_t i = lane; i < k; i += 64) {
                L.keys[from + i] = dev_load(&cl.s->keys[c * cap + i]);
                L.ids[from + i] = dev_load(&cl.s->ids[c * cap + i]);
            }
        }
        if (tid == 0) L.n = n;
        __syncthreads();
    }
    return true;
}

// rank-th and rank1-th largest (1-based) of the n <= ST keys in L.gmax, n a multiple of 4; 0 where n is smaller.  Whole
// workgroup; results in L.bound, L.bound1.
__device__ __forceinline__ void kth_of_groups(ShortLds &L, int n, int rank, int rank1, int tid)
{
    if (tid == 0) L.bound = L.bound1 = 0;
    __syncthreads();
    if (tid < n) {
        const uint32_t mine = L.gmax[tid];
        int above = 0, equal = 0;
        for (int i = 0; i < n; i += 4) {
            const u32x4 o = *reinterpret_cast<const u32x4 *>(&L.gmax[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e) { above += o[e] > mine; equal += o[e] == mine; }
        }
        if (above < rank && rank <= above + equal) L.bound = mine;   // all writers hold the same key
        if (above < rank1 && rank1 <= above + equal) L.bound1 = mine;
    }
    __syncthreads();
}

enum { SHORT_DONE = 1, SHORT_GENERAL = 0, SHORT_LOST = -1 };

// What the short path found out about a row that it leaves to the general path.
struct Known {
    uint32_t kmax = 0;             // key of the maximum, if it is finite; else 0
    uint32_t bound = 0;            // top-k: a lower bound of the selection's last key; 0: none
    int bin = -1;                  // top-p without top-k: the bin of the nucleus' last token, with
    uint64_t above = 0, target = 0;   // the mass above that bin and the nucleus' mass
};

// Bin of a token that has any mass: 1/16 octave of weight, 0 at the maximum, below 497 (weights above 2^-31).
__device__ __forceinline__ int fine_bin(const RowCtx &r, float x) { return (int)((r.mx - x) * r.scale * 16.f); }

// One row.  zs: this workgroup's ids [seg_lo, seg_lo + Vs) of the row z; top_k at most SHORT_K_MAX.  Every workgroup of the
// cluster returns the same.
__device__ __forceinline__ int short_row(ShortLds &L, Cluster &cl, const float *z, int V, int seg_lo, int seg_len, int Vs, bool vec4, float scale, int top_k,
                         float top_p, float uniform, int32_t *out, int32_t *err, Known &known)
{
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const bool use_k = top_k > 0 && top_k < V, nucleus = top_p < 1.f;
    const float *zs = z + seg_lo;

    // ---- pass 1: the maximum, (top-k) maxima per group of threads, (top-p) the minimum ----
    uint32_t kmax = 0, kmin = 0xFFFFFFFFu;
    if (use_k || !nucleus)
        for_whole_row(zs, Vs, vec4, tid, [&](int, float x, bool ok) { if (ok) kmax = max(kmax, order_key(x)); });
    else
        for_whole_row(zs, Vs, vec4, tid, [&](int, float x, bool ok) {
            if (ok) { kmax = max(kmax, order_key(x)); kmin = min(kmin, order_key(x)); }
        });
    L.gmax[tid] = kmax;
    if (tid == 0) L.n = 0;
    if (!use_k && nucleus)
        for (int i = tid; i < FINE_COPIES * FINE_BINS; i += ST) (&L.fine[0][0])[i] = 0;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off));
    }
    if (lane == 0) L.red[wave] = (uint64_t)kmin << 32 | kmax;
    __syncthreads();
    kmax = (uint32_t)L.red[lane & 15];
    kmin = (uint32_t)(L.red[lane & 15] >> 32);
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
        kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off));
    }
    uint32_t bound = 0;
    if (use_k) {
        int groups = ST;
        if (top_k <= 64) {   // 256 groups rank four times faster than 1024, and top_k of them still bound tightly
            groups = 256;
            uint32_t m = tid < 256 ? max(max(L.gmax[tid], L.gmax[tid + 256]), max(L.gmax[tid + 512], L.gmax[tid + 768])) : 0;
            __syncthreads();
            if (tid < 256) L.gmax[tid] = m;
            __syncthreads();
        }
        // With C workgroups: at least top_k tokens reach the smallest of the workgroups' ceil(top_k / C)-th largest, too.
        kth_of_groups(L, groups, top_k, (top_k + cl.C - 1) / cl.C, tid);
        bound = L.bound;
        if (cl.C > 1 && tid == 0) { dev_store(&cl.s->bound_k[cl.c], bound); dev_store(&cl.s->bound_1[cl.c], L.bound1); }
    }
    if (cl.C > 1) {
        if (tid == 0) { dev_store(&cl.s->kmax[cl.c], kmax); dev_store(&cl.s->kmin[cl.c], kmin); }
        if (!cluster_sync(cl, err)) return SHORT_LOST;
        uint32_t lo1 = 0xFFFFFFFFu;
        if (lane < cl.C) {
            kmax = dev_load(&cl.s->kmax[lane]);
            kmin = dev_load(&cl.s->kmin[lane]);
            if (use_k) { bound = dev_load(&cl.s->bound_k[lane]); lo1 = dev_load(&cl.s->bound_1[lane]); }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off));
            kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off));
            bound = max(bound, (uint32_t)__shfl_xor((int)bound, off));
            lo1 = min(lo1, (uint32_t)__shfl_xor((int)lo1, off));
        }
        if (use_k) bound = max(bound, lo1);
    }
    // +inf or NaN, or nothing above -inf; or a temperature so small that the scale overflows: the maximum's own weight is
    // then exp2(0 * inf), no token has any mass, and the general path answers with the arg-max
    if (kmax >= 0xFF800000u || kmax <= 0x007FFFFFu || scale == INFINITY) return SHORT_GENERAL;
    RowCtx r{z, V, key_logit(kmax), scale};
    known.kmax = kmax;
    known.bound = bound;

    if (use_k) {
        // ---- pass 2: the tokens at or above the bound; the first workgroup does the rest ----
        for_whole_row<true>(zs, Vs, vec4, tid, [&](int i, float x, bool ok) {
            const uint32_t key = order_key(x);
            list_push(L, ok && key >= bound, key, seg_lo + i, lane);
        }, [&] { return __builtin_amdgcn_readfirstlane(*(volatile uint32_t *)&L.n) <= LIST_K_MAX; });
        list_publish(L, cl, tid);
        if (cl.C > 1) { if (!cluster_sync(cl, err)) return SHORT_LOST; }
        else __syncthreads();
        if (!list_gather(L, cl, LIST_K_MAX, tid)) return SHORT_GENERAL;
        if (cl.c != 0) return SHORT_DONE;
        const int n = (int)L.n;
        const uint32_t key = tid < n ? L.keys[tid] : 0, id = tid < n ? L.ids[tid] : 0;
        int rank = 0;   // in order O
        if (tid < n)
            for (int i = 0; i < n; i += 4) {   // entries past n are masked out
                const u32x4 k4 = *reinterpret_cast<const u32x4 *>(&L.keys[i]), i4 = *reinterpret_cast<const u32x4 *>(&L.ids[i]);
#pragma unroll
                for (int e = 0; e < 4; ++e) rank += i + e < n && (k4[e] > key || (k4[e] == key && i4[e] < id));
            }
        const uint64_t mine = tid < n && rank < top_k ? fix_mass(r, key_logit(key)) : 0;   // 0: not in S_k
        // L.sub: masses of S_k by rank, then of S by position in the list (n <= 1024 = MAX_SUB)
        L.sub[tid] = 0;
        __syncthreads();
        if (tid < n && rank < top_k) L.sub[rank] = mine;
        __syncthreads();
        bool member = tid < n && rank < top_k;
        if (nucleus) {
            uint64_t tot = 0, before = 0;
            for (int i = 0; i < min(n, top_k); ++i) {
                const uint64_t m = L.sub[i];
                tot += m;
                if (i < rank) before += m;
            }
            uint64_t target = (uint64_t)((double)top_p * (double)tot);
            if (target < 1) target = 1;
            if (target > tot) target = tot;
            member = member && before < target;   // the shortest prefix of O that reaches the target
        }
        __syncthreads();
        if (tid < n) L.sub[tid] = member ? mine : 0;
        __syncthreads();
        if (tid < n) {
            uint64_t tot = 0, before = 0;         // of S; of its tokens with a lower id
            for (int i = 0; i < n; ++i) {
                const uint64_t m = L.sub[i];
                tot += m;
                if (L.ids[i] < id) before += m;
            }
            uint64_t target = (uint64_t)((double)uniform * (double)tot);
            if (target >= tot) target = tot ? tot - 1 : 0;
            const uint64_t m = L.sub[tid];
            if (m && before <= target && target < before + m) *out = (int32_t)id;
        }
        return SHORT_DONE;
    }

    // ---- pass 2: masses by bin ----
    int bin = 0x7FFFFFFF;   // no nucleus: every token counts as above the bin, and the list stays empty
    uint64_t target = 0;
    if (nucleus) {
        // So many tokens on so few bins that the last one's list would overflow: a quarter of LIST_MAX per bin on average
        // are LIST_MAX in the middle of a normal distribution.
        if ((float)V > ((r.mx - key_logit(kmin)) * r.scale * 16.f + 1.f) * (LIST_MAX / 4)) return SHORT_GENERAL;
        uint64_t sum = 0;
        for_whole_row<true>(zs, Vs, vec4, tid, [&](int, float x, bool ok) {
            const uint64_t m = ok ? fix_mass(r, x) : 0;
            if (m) atomicAdd((unsigned long long *)&L.fine[lane & (FINE_COPIES - 1)][fine_bin(r, x)], (unsigned long long)m);
            sum += m;
        });
        sum = wave_sum(sum);
        __syncthreads();
        if (lane == 0) L.red[wave] = sum;
        uint64_t mine = 0;
        if (tid < FINE_BINS)
    #pragma unroll
            for (int k = 0; k < FINE_COPIES; ++k) mine += L.fine[k][tid];
        __syncthreads();
        sum = 0;
        for (int w = 0; w < 16; ++w) sum += L.red[w];
        if (cl.C > 1) {
            if (tid < FINE_BINS && mine) __hip_atomic_fetch_add((unsigned long long *)&cl.s->fine[tid], (unsigned long long)mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (tid == 0) dev_store(&cl.s->mass[cl.c], sum);
            if (!cluster_sync(cl, err)) return SHORT_LOST;
            if (tid < FINE_BINS) mine = dev_load(&cl.s->fine[tid]);
            sum = wave_sum(lane < cl.C ? dev_load(&cl.s->mass[lane]) : (uint64_t)0);
        }
        if (tid < FINE_BINS) L.fine[0][tid] = mine;
        __syncthreads();
        target = (uint64_t)((double)top_p * (double)sum);
        if (target < 1) target = 1;
        if (target > sum) target = sum;
        if (wave == 0) {   // lane l owns bins 8l .. 8l+7; bin 0 holds the largest logits
            uint64_t v[8], own = 0;
    #pragma unroll
            for (int e = 0; e < 8; ++e) { v[e] = L.fine[0][8 * lane + e]; own += v[e]; }
            uint64_t pre = own;
    #pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint64_t o = __shfl_up(pre, off);
                if (lane >= off) pre += o;
            }
            pre -= own;   // mass of the bins before this lane's
            if (pre < target && target <= pre + own) {
                uint64_t a = pre;
                int e = 0;
                while (e < 7 && a + v[e] < target) a += v[e++];
                L.bin = 8 * lane + e;
                L.above = a;
            }
        }
        __syncthreads();
        bin = L.bin;
        known.bin = bin;
        known.above = L.above;
        known.target = target;
        // at least so many tokens: none of the bin's weights is above exp2(-bin / 16)
        if ((float)L.fine[0][bin] > (LIST_MAX * 1.001f) * 2147483648.f * __builtin_amdgcn_exp2f(bin * -0.0625f)) return SHORT_GENERAL;
    }

    // ---- pass 3: sums per batch of the tokens above the bin, and the bin's own tokens ----
    // Same geometry in every workgroup: wave w of workgroup c owns ids [w * per, w * per + per) of its segment.
    const int per = ((min(seg_len, V) + 15) / 16 + 3) & ~3;
    const int n_batch = (per + 64 * SU - 1) / (64 * SU);
    const int lo = min(Vs, wave * per), hi = min(Vs, lo + per);
    auto visit = [&](int i, float x, bool ok) -> uint64_t {
        const uint64_t m = ok ? fix_mass(r, x) : 0;
        const int b = fine_bin(r, x);
        list_push(L, m != 0 && b == bin, order_key(x), seg_lo + i, lane);
        return m != 0 && b < bin ? m : 0;
    };
    constexpr int NB = 4;   // batches whose loads are in flight together
    for (int b0 = 0; b0 < n_batch; b0 += NB) {
        float x[NB][SU];
#pragma unroll
        for (int bb = 0; bb < NB; ++bb)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int at = lo + (b0 + bb) * 64 * SU + h * 256 + 4 * lane;
                if (vec4) {
                    const f32x4 t = at < hi ? *reinterpret_cast<const f32x4 *>(zs + at) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[bb][4 * h + e] = t[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[bb][4 * h + e] = at + e < hi ? zs[at + e] : 0.f;
                }
            }
#pragma unroll
        for (int bb = 0; bb < NB; ++bb) {
            if (b0 + bb >= n_batch) break;
            uint64_t s = 0;
#pragma unroll
            for (int e = 0; e < SU; ++e) {
                const int at = lo + (b0 + bb) * 64 * SU + (e >> 2) * 256 + 4 * lane + (e & 3);
                s += visit(at, x[bb][e], at < hi);
            }
            if (__ballot(s != 0)) s = wave_sum(s);
            if (lane == 0) L.sub[wave * n_batch + b0 + bb] = s;
        }
    }
    __syncthreads();
    const int n_sub = cl.C * 16 * n_batch;   // <= MAX_SUB (launch_sample_rows)
    if (cl.C > 1) {
        for (int i = tid; i < 16 * n_batch; i += ST) dev_store(&cl.s->sub[cl.c * 16 * n_batch + i], L.sub[i]);
        if (nucleus) list_publish(L, cl, tid);
        if (!cluster_sync(cl, err)) return SHORT_LOST;
        if (tid < n_sub) L.sub[tid] = dev_load(&cl.s->sub[tid]);   // the whole row's sums, one per thread at most
    }
    if (nucleus && !list_gather(L, cl, LIST_MAX, tid)) return SHORT_GENERAL;
    const int n = (int)L.n;

    // The first workgroup has everything; without a list to look through, each finds the draw and its owner finishes.
    if (nucleus && cl.c != 0) return SHORT_DONE;

    // ---- the last token of S inside the list: radix select on masses, then, if S takes its ties only in part, on ids ----
    uint32_t key_b = 0, id_b = 0xFFFFFFFFu;   // S: keys above key_b, and those equal to it with an id up to id_b
    if (nucleus) {
        auto select = [&](auto &&digits, auto &&value, uint64_t want, uint64_t above) -> uint32_t {   // leaves the sum above in L.above
            uint32_t prefix = 0;
            for (int d = 3; d >= 0; --d) {
                if (tid < 256) L.bins[tid] = 0;
                __syncthreads();
                for (int i = tid; i < n; i += ST) {
                    const uint32_t x = digits(i);
                    if (d == 3 || (x >> (8 * (d + 1))) == prefix)
                        atomicAdd((unsigned long long *)&L.bins[(x >> (8 * d)) & 255u], (unsigned long long)value(i));
                }
                __syncthreads();
                if (wave == 0) {
                    uint64_t higher;
                    const int g = pick_bin<uint64_t>(L.bins, want, above, higher, lane);
                    if (lane == 0) { L.prefix = (prefix << 8) | (uint32_t)g; L.above = above + higher; L.equal = L.bins[g]; }
                }
                __syncthreads();
                prefix = L.prefix;
                above = L.above;
            }
            return prefix;
        };
        key_b = select([&](int i) { return L.keys[i]; }, [&](int i) { return fix_mass(r, key_logit(L.keys[i])); }, target, L.above);
        const uint64_t mass_b = fix_mass(r, key_logit(key_b));   // not zero: a token of the list
        const uint64_t all = L.equal;                            // mass of the tokens with exactly this key
        const uint64_t n_b = (target - L.above + mass_b - 1) / mass_b;   // how many of them S takes, lowest ids first; at least one
        if (n_b * mass_b < all)
            id_b = ~select([&](int i) { return ~L.ids[i]; }, [&](int i) { return (uint64_t)(L.keys[i] == key_b); }, n_b, 0);
        for (int i = tid; i < n; i += ST) {
            const uint32_t key = L.keys[i], id = L.ids[i];
            if (key > key_b || (key == key_b && id <= id_b)) {
                const int c = (int)id / seg_len, at = (int)id - c * seg_len;
                atomicAdd((unsigned long long *)&L.sub[(c * 16 + at / per) * n_batch + at % per / (64 * SU)],
                          (unsigned long long)fix_mass(r, key_logit(key)));
            }
        }
    }
    __syncthreads();
    // ---- the batch that holds the draw, then the token in it ----
    if (wave != 0) return SHORT_DONE;
    uint64_t own = 0;
    const int chunk = (n_sub + 63) / 64;   // <= 16 sums per lane
    for (int e = 0; e < chunk; ++e) own += lane * chunk + e < n_sub ? L.sub[lane * chunk + e] : 0;
    uint64_t pre = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t o = __shfl_up(pre, off);
        if (lane >= off) pre += o;
    }
    const uint64_t tot = __shfl(pre, 63);
    pre -= own;
    uint64_t t = (uint64_t)((double)uniform * (double)tot);
    if (t >= tot) t = tot ? tot - 1 : 0;
    const uint64_t holder = __ballot(own && pre <= t && t < pre + own);
    const int src = holder ? __ffsll((long long)holder) - 1 : 0;
    int batch = lane * chunk;
    if (lane == src)
        for (int e = 0; e < chunk - 1 && pre + L.sub[batch] <= t; ++e) pre += L.sub[batch++];
    batch = __shfl(batch, src);
    t -= __shfl(pre, src);                 // offset of the draw inside the batch
    const int seg = batch / (16 * n_batch), w = batch / n_batch % 16;
    if (!nucleus && cl.C > 1 && seg != cl.c) return SHORT_DONE;
    const int seg_at = seg * seg_len, seg_end = min(V, seg_at + seg_len);
    const int wave_end = min(seg_end, seg_at + (w + 1) * per);
    const int b_lo = seg_at + w * per + batch % n_batch * 64 * SU, b_hi = min(wave_end, b_lo + 64 * SU);
    uint64_t carry = 0;
    int found = 0;
    bool open = true;
    for_row(z, b_lo, b_hi, lane, 64, [&](int i, float x, bool ok) {
        if (!open) return;                 // wave-uniform
        const uint32_t key = order_key(x);
        const uint64_t m = ok && (key > key_b || (key == key_b && (uint32_t)i <= id_b)) ? fix_mass(r, x) : 0;
        uint64_t inc = m;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t o = __shfl_up(inc, off);
            if (lane >= off) inc += o;
        }
        const uint64_t hit = __ballot(m > 0 && carry + inc > t);
        if (hit) { found = i - lane + __ffsll((long long)hit) - 1; open = false; }
        carry += __shfl(inc, 63);
    });
    if (lane == 0) *out = found;
    return SHORT_DONE;
}

// One row, by the workgroups of a cluster (or one workgroup): the row's token to sampled[row].
template <bool SHORT>
__device__ __forceinline__ void sample_row(Cluster &cl, const float *logits, int row, int V, float inv_temperature, int top_k, float top_p,
                                           const float *uniforms, int32_t *sampled, int32_t *err)
{
    __shared__ uint32_t chist[256];
    __shared__ uint64_t mhist[256];
    __shared__ float red_f[16];
    __shared__ uint32_t red_c[16];
    __shared__ uint32_t sh_prefix, sh_need, sh_count_b;
    __shared__ uint64_t sh_above, sh_target;
    __shared__ int sh_wave, sh_batch, sh_token;
    __shared__ uint64_t sub[16][MAX_BATCH];   // mass of S per (wave, batch of 512 ids)
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, C = cl.C;
    // this workgroup's token ids: [seg_lo, seg_hi), whole groups of four so that 16-byte loads stay aligned
    const int seg_len = ((V + C - 1) / C + 3) & ~3;
    const int seg_lo = min(V, cl.c * seg_len), seg_hi = min(V, seg_lo + seg_len), Vs = seg_hi - seg_lo;
    RowCtx r;
    r.z = logits + (size_t)row * V;
    r.V = V;
    const float *zs = r.z + seg_lo;   // the segment
    auto give_up = [&]() { if (cl.c == 0 && tid == 0) sampled[row] = -1; };
    // The scratch's bins start at zero; a barrier (of the maxima) comes before anything is added to them.
    if (C > 1) {
        uint32_t *w = &cl.s->chist[0][0];
        constexpr int WORDS = HIST_PASSES * 256 * 3;
        for (int i = cl.c * ST + tid; i < WORDS; i += C * ST) __hip_atomic_store(w + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int i = cl.c * ST + tid; i < FINE_BINS; i += C * ST) dev_store(&cl.s->fine[i], (uint64_t)0);
    }

    const bool vec4 = (V & 3) == 0 && (reinterpret_cast<uintptr_t>(r.z) & 15) == 0;
    Known known;
    if (SHORT) {
        __shared__ ShortLds short_lds;
        const int done = short_row(short_lds, cl, r.z, V, seg_lo, seg_len, Vs, vec4, 1.4426950408889634f * inv_temperature, top_k, top_p,
                                   uniforms[row], sampled + row, err, known);
        if (done == SHORT_LOST) give_up();
        if (done != SHORT_GENERAL) return;
    }

    // ---- max ----
    float mx = key_logit(known.kmax);
    if (!SHORT || !known.kmax) {
        mx = -INFINITY;
        for_whole_row(zs, Vs, vec4, tid, [&](int, float z, bool ok) { if (ok) mx = fmaxf(mx, z); });
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        if (lane == 0) red_f[wave] = mx;
        __syncthreads();
        mx = red_f[0];
        for (int w = 1; w < 16; ++w) mx = fmaxf(mx, red_f[w]);
        __syncthreads();
        if (C > 1) {
            if (tid == 0) __hip_atomic_store(&cl.s->gmax[cl.c], mx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!cluster_sync(cl, err)) { give_up(); return; }
            for (int w = 0; w < C; ++w) mx = fmaxf(mx, __hip_atomic_load(&cl.s->gmax[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
    }
    r.mx = mx;
    r.scale = 1.4426950408889634f * inv_temperature;

    // ---- top-k: key_a = key of the top_k-th token of O, n_a = how many tokens with exactly that key are kept ----
    uint32_t key_a = 0, n_a = 0, total_a = 0;   // total_a: tokens of the row with key == key_a
    const bool use_k = top_k > 0 && top_k < V;
    bool lost = false;
    if (use_k) {
        uint32_t prefix = 0, need = (uint32_t)top_k;
        int first = 3;   // leading digits that every key from the bound to the maximum has are known
        if (SHORT && known.bound) first = common_digits(known.bound, known.kmax, prefix);
        for (int d = first; d >= 0 && !lost; --d) {
            if (tid < 256) chist[tid] = 0;
            __syncthreads();
            BinRun run{0, 0, 0, false};
            for_whole_row(zs, Vs, vec4, tid, [&](int, float z, bool ok) {
                const uint32_t key = order_key(z);
                if (ok && (d == 3 || (key >> (8 * (d + 1))) == prefix)) run_add(run, (key >> (8 * d)) & 255u, 0, chist, nullptr);
            });
            run_flush(run, chist, nullptr);
            __syncthreads();
            if (!merge_bins(cl, 3 - d, chist, nullptr, true, false, tid, err)) { lost = true; break; }
            if (wave == 0) {
                uint32_t higher;
                const int g = pick_bin<uint32_t>(chist, need, 0u, higher, lane);
                if (lane == 0) {
                    sh_prefix = (prefix << 8) | (uint32_t)g;
                    sh_need = need - higher;
                    sh_count_b = chist[g];   // after the last digit: every token of the row with exactly this key
                }
            }
            __syncthreads();
            prefix = sh_prefix;
            need = sh_need;
            __syncthreads();
        }
        key_a = prefix;   // the key of the k-th token
        n_a = need;       // 1 <= n_a <= total_a
        total_a = sh_count_b;
        __syncthreads();
    }
    if (lost) { give_up(); return; }

    // the n_a kept tokens at the top-k threshold all carry the same logit, hence the same mass
    uint64_t mass_a = 0;
    if (use_k) {
        const uint32_t u = (key_a & 0x80000000u) ? (key_a & 0x7FFFFFFFu) : ~key_a;   // invert order_key
        mass_a = fix_mass(r, bits_f32(u));
    }

    // ---- top-p: key_b = key of the last token of S, n_b = how many tokens with exactly that key are in S.
    // The first pass's bins add up to Z_k, from which the target mass follows. ----
    uint32_t key_b = key_a, n_b = n_a;
    uint32_t count_b = n_a;   // kept tokens with key == key_b
    uint32_t total_b = total_a;   // tokens of the row with key == key_b
    {
        const bool nucleus = top_p < 1.f;
        const bool in_bin = SHORT && known.bin >= 0;   // only the tokens of one bin are left to look through
        uint64_t target = in_bin ? known.target : 0, above = in_bin ? known.above : 0;
        uint32_t prefix = 0;
        int first = 3;
        if (in_bin) {
            // logits of the bin, a hundredth of a bin and a few units of rounding wider than it is
            const float width = 1.f / (16.f * r.scale), slack = fabsf(r.mx) * 1e-6f;
            const float low = r.mx - ((float)known.bin + 1.01f) * width - slack, high = r.mx - ((float)known.bin - 0.01f) * width + slack;
            if (low > -INFINITY && high < INFINITY) first = common_digits(order_key(low), order_key(high), prefix);
        } else if (SHORT && use_k && known.kmax) {
            first = common_digits(key_a, known.kmax, prefix);
        }
        for (int d = first; nucleus && d >= 0 && !lost; --d) {
            if (tid < 256) { mhist[tid] = 0; chist[tid] = 0; }
            __syncthreads();
            BinRun run{0, 0, 0, false};
            uint32_t *cbins = d == 0 ? chist : nullptr;   // counts matter only for the exact key (the ties at key_b)
            auto look = [&](auto &&mass_of) {
                for_whole_row(zs, Vs, vec4, tid, [&](int, float z, bool ok) {
                    const uint32_t key = order_key(z);
                    if (ok && (!use_k || key > key_a) && (d == 3 || (key >> (8 * (d + 1))) == prefix))
                        run_add(run, (key >> (8 * d)) & 255u, mass_of(z), cbins, mhist);
                });
            };
            if (in_bin) look([&](float z) { return fine_bin(r, z) == known.bin ? fix_mass(r, z) : 0ull; });
            else look([&](float z) { return fix_mass(r, z); });
            run_flush(run, cbins, mhist);
            // the kept tokens at the top-k threshold are added once per row, by the cluster's first workgroup
            if (tid == 0 && cl.c == 0 && use_k && (d == 3 || (key_a >> (8 * (d + 1))) == prefix)) {
                const uint32_t g = (key_a >> (8 * d)) & 255u;
                atomicAdd((unsigned long long *)&mhist[g], (unsigned long long)n_a * mass_a);
                atomicAdd(&chist[g], n_a);
            }
            __syncthreads();
            if (!merge_bins(cl, 4 + (3 - d), chist, mhist, d == 0, true, tid, err)) { lost = true; break; }
            if (wave == 0) {
                if (d == first && !in_bin) {   // Z_k = the sum of all bins; the nucleus target follows from it
                    uint64_t tot = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) tot += mhist[4 * lane + e];
#pragma unroll
                    for (int off = 32; off >= 1; off >>= 1) tot += __shfl_xor(tot, off);
                    target = (uint64_t)((double)top_p * (double)tot);
                    if (target < 1) target = 1;
                    if (target > tot) target = tot;
                    if (lane == 0) sh_target = target;
                }
                if (nucleus) {
                    uint64_t higher;
                    const int g = pick_bin<uint64_t>(mhist, target, above, higher, lane);
                    if (lane == 0) {
                        sh_prefix = (prefix << 8) | (uint32_t)g;
                        sh_above = above + higher;
                        sh_count_b = chist[g];
                    }
                }
            }
            __syncthreads();
            if (!in_bin) target = sh_target;
            if (nucleus) {
                prefix = sh_prefix;
                above = sh_above;
            }
            __syncthreads();
        }
        if (nucleus && !lost) {
            key_b = prefix;
            count_b = sh_count_b;   // after the last digit: kept tokens with exactly this key
            const uint32_t ub = (key_b & 0x80000000u) ? (key_b & 0x7FFFFFFFu) : ~key_b;
            const uint64_t mass_b = fix_mass(r, bits_f32(ub));
            uint64_t nb = mass_b ? (target - above + mass_b - 1) / mass_b : 1;
            if (nb < 1) nb = 1;
            if (nb > count_b) nb = count_b;
            n_b = (uint32_t)nb;
            total_b = (use_k && key_b == key_a) ? total_a : count_b;
        }
    }
    if (lost) { give_up(); return; }
    const bool all_kept = !use_k && !(top_p < 1.f);   // S is the whole vocabulary

    // ---- sample in token-id order.  Wave w of this workgroup owns ids [lo, hi) of the segment; lanes stride by 64. ----
    const int per = (Vs + 15) / 16;
    const int lo = seg_lo + min(Vs, wave * per), hi = min(seg_hi, lo + per);
    // (1) ties at key_b below each wave, so that "the n_b lowest ids" is decidable per element
    uint32_t ties = 0;
    const bool partial_ties = !all_kept && n_b < total_b;   // else every tie is a member: no ranks needed
    if (partial_ties)
        for_row(r.z, lo, hi, lane, 64, [&](int, float z, bool ok) {
            ties += (uint32_t)__popcll(__ballot(ok && order_key(z) == key_b));
        });
    if (lane == 0) red_c[wave] = ties;
    __syncthreads();
    uint32_t tie_base = 0;
    for (int w = 0; w < wave; ++w) tie_base += red_c[w];
    if (C > 1 && partial_ties) {   // ties in the workgroups before this one
        uint32_t mine = 0;
        for (int w = 0; w < 16; ++w) mine += red_c[w];
        if (tid == 0) __hip_atomic_store(&cl.s->gties[cl.c], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!cluster_sync(cl, err)) { give_up(); return; }
        for (int w = 0; w < cl.c; ++w) tie_base += __hip_atomic_load(&cl.s->gties[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // (2) mass of S inside each wave
    auto member_mass = [&](float z, bool in_range, uint32_t &tie_seen) -> uint64_t {   // wave-uniform call; updates the running tie count
        const uint32_t key = order_key(z);
        const bool tie = in_range && !all_kept && key == key_b;
        uint32_t rank = 0;
        if (partial_ties) {
            const uint64_t bal = __ballot(tie);
            rank = tie_seen + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
            tie_seen += (uint32_t)__popcll(bal);
        }
        const bool member = in_range && (all_kept || key > key_b || (tie && rank < n_b));
        return member ? fix_mass(r, z) : 0ull;
    };
    // One entry per batch of 8 x 64 consecutive ids of every wave: the target is then located in one
    // batch instead of a walk through the wave's whole range.
    if (lane < MAX_BATCH) sub[wave][lane] = 0;   // ranges past the vocabulary leave their entries at zero
    {
        uint32_t seen = tie_base;
        uint64_t bsum = 0;
        int calls = 0, calls_total = 0;
        for_row(r.z, lo, hi, lane, 64, [&](int, float z, bool ok) {
            bsum += member_mass(z, ok, seen);
            if (++calls == SU) {
                uint64_t t = bsum;
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
                const int batch = (calls_total++);
                if (lane == 0) sub[wave][batch] = t;
                calls = 0;
                bsum = 0;
            }
        });
    }
    __syncthreads();
    // (3) the (workgroup, wave, batch) whose id range holds the target, then the element inside it
    const int n_batch = (per + 64 * SU - 1) / (64 * SU);
    uint64_t wg_before = 0, row_total = 0;   // member mass in the workgroups before this one / in the whole row
    if (C > 1) {
        uint64_t mine = 0;
        if (tid == 0)
            for (int w = 0; w < 16; ++w)
                for (int bt = 0; bt < n_batch; ++bt) mine += sub[w][bt];
        if (tid == 0) __hip_atomic_store((unsigned long long *)&cl.s->gsub[cl.c], (unsigned long long)mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!cluster_sync(cl, err)) { give_up(); return; }
        for (int w = 0; w < C; ++w) {
            const uint64_t m = __hip_atomic_load((unsigned long long *)&cl.s->gsub[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (w < cl.c) wg_before += m;
            row_total += m;
        }
    }
    if (tid == 0) {
        uint64_t tot = 0;
        for (int w = 0; w < 16; ++w)
            for (int bt = 0; bt < n_batch; ++bt) tot += sub[w][bt];
        const uint64_t mine = tot;
        if (C > 1) tot = row_total;
        // the draw uses this recomputed total, so that it always lands inside S
        const double u = (double)uniforms[row];
        uint64_t target = (uint64_t)(u * (double)tot);
        if (target >= tot) target = tot ? tot - 1 : 0;
        // the workgroup whose ids hold the target walks on; with no mass at all the last one answers
        const bool here = C == 1 || (tot ? (target >= wg_before && target < wg_before + mine) : cl.c == C - 1);
        target -= here ? wg_before : 0;
        uint64_t acc = 0;
        int w = 0, bt = 0;
        bool done = false;
        for (w = 0; w < 16 && !done; ++w)
            for (bt = 0; bt < n_batch; ++bt) {
                if (acc + sub[w][bt] > target) { done = true; break; }
                acc += sub[w][bt];
            }
        if (done) --w; else { w = 15; bt = n_batch > 0 ? n_batch - 1 : 0; }   // an empty range walks nothing and falls through to the arg-max
        sh_wave = here ? w : -1;
        sh_batch = bt;
        sh_above = target - acc;   // offset of the target inside that batch
        sh_token = -1;
    }
    __syncthreads();
    if (wave == sh_wave) {
        const uint64_t target = sh_above;
        const int b_lo = lo + sh_batch * 64 * SU, b_hi = min(hi, b_lo + 64 * SU);
        // ties before this batch inside the wave's range (only needed when ties are taken partially)
        uint32_t seen = tie_base;
        if (partial_ties)
            for_row(r.z, lo, b_lo, lane, 64, [&](int, float z, bool ok) {
                seen += (uint32_t)__popcll(__ballot(ok && order_key(z) == key_b));
            });
        uint64_t carry = 0;
        int found = -1;
        int last_member = -1;
        for_row(r.z, b_lo, b_hi, lane, 64, [&](int i, float z, bool ok) {
            if (found >= 0) return;                     // wave-uniform
            const int base = i - lane;
            const uint64_t m = member_mass(z, ok, seen);
            uint64_t inc = m;   // inclusive scan over lanes
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint64_t o = __shfl_up(inc, off);
                if (lane >= off) inc += o;
            }
            const bool hit = m > 0 && carry + inc > target;
            const uint64_t hb = __ballot(hit);
            const uint64_t mb = __ballot(m > 0);
            if (mb) last_member = base + 63 - __clzll(mb);
            if (hb) found = base + __ffsll((long long)hb) - 1;
            carry += __shfl(inc, 63);
        });
        if (lane == 0) sh_token = found >= 0 ? found : last_member;
    }
    __syncthreads();
    if (tid == 0 && sh_wave >= 0) {
        int t = sh_token;
        if (t < 0) {   // no mass at all in the chosen range (cannot happen with finite logits): the arg-max
            t = 0;
            for (int i = 1; i < V; ++i)
                if (r.z[i] > r.z[t]) t = i;
        }
        sampled[row] = t;
    }
}

// grid = rows * C workgroups of 1024 threads, cluster g on row g.  A cluster takes one row only: most of its workgroups are
// done while the first still reads their scratch, which nobody may clear for another row then.
template <bool SHORT>
__global__ __launch_bounds__(ST) void sample_rows_kernel(const float *logits, int V, float inv_temperature, int top_k, float top_p,
                                                         const float *uniforms, int32_t *sampled, int C, SampleScratch *scratch,
                                                         int32_t *err)
{
    const int row = blockIdx.x / C;
    Cluster cl{C > 1 ? scratch + row : nullptr, C, (int)(blockIdx.x % C), 0u, false};
    sample_row<SHORT>(cl, logits, row, V, inv_temperature, top_k, top_p, uniforms, sampled, err);
    // Leave the counters at zero for the next launch on this scratch (a cluster that gave up leaves them as
    // they are: the launcher's caller learns of it through *err and clears the scratch).
    if (C > 1 && !cl.failed && threadIdx.x == 0) {
        const uint32_t old = __hip_atomic_fetch_add(&cl.s->departures, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (old == (uint32_t)C - 1) {
            __hip_atomic_store(&cl.s->arrivals, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&cl.s->departures, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// Zeroes the clusters' two counters; everything else in the scratch is written before it is read (a kernel, not a memset:
// the launch may be captured in a graph).
__global__ void sample_scratch_clear_kernel(SampleScratch *s, int rows)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) s[i].arrivals = s[i].departures = 0u;
}

}  // namespace

// Workgroups per row for a launch of `rows` rows on a device of n_cu compute units: the largest power of two
// (at most 16) that keeps the whole grid resident at one workgroup per compute unit; 1 without scratch.
static int sample_cluster_size(int rows, int n_cu)
{
    int c = 1;
    while (c * 2 <= MAX_CLUSTER && (long)rows * (c * 2) <= n_cu) c *= 2;
    return c;
}

size_t sample_scratch_bytes(int rows, int n_cu)
{
    const int c = sample_cluster_size(rows, n_cu);
    return c > 1 ? (size_t)rows * sizeof(SampleScratch) : 0;
}

hipError_t launch_sample_rows(const float *logits, int rows, int V, float temperature, int top_k, float top_p,
                              const float *uniforms, int32_t *sampled, void *scratch, size_t scratch_bytes, bool scratch_clean, int n_cu,
                              int32_t *err, hipStream_t s)
{
    if ((long)V > 16L * MAX_BATCH * 64 * SU) return hipErrorInvalidValue;
    int C = scratch ? sample_cluster_size(rows, n_cu > 0 ? n_cu : 256) : 1;
    if (C > 1 && scratch_bytes < (size_t)rows * sizeof(SampleScratch)) C = 1;
    if (C > 1 && (long)(V / C) > (long)MAX_BATCH * 16 * 64 * SU) return hipErrorInvalidValue;
    if (C > 1 && !scratch_clean) {
        hipLaunchKernelGGL(sample_scratch_clear_kernel, dim3((rows + 63) / 64), dim3(64), 0, s, (SampleScratch *)scratch, rows);
    }
    hipLaunchKernelGGL((top_k > SHORT_K_MAX && top_k < V ? sample_rows_kernel<false> : sample_rows_kernel<true>), dim3(rows * C), dim3(ST), 0, s, logits, V, 1.f / temperature, top_k, top_p, uniforms,
                       sampled, C, (SampleScratch *)scratch, err);
    return hipGetLastError();
}
