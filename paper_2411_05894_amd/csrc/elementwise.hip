// Small bandwidth-trivial kernels around the GEMMs: token/length validation with the
// embedding gather (which also writes the first layer's packed operands and sums of
// squares), arg-max merge + greedy prefix acceptance, rollback, cache import/export,
// weight reordering at init, and the packing helpers of the kernel-level entry points.
// None of them is in the paper's Table 2 (it lists the matrix operations only); they move
// O(M*h) bytes against O(params) for the GEMMs.
#include "kernels.h"

namespace {

// Room for the k + 1 new rows behind len cached ones (max_seq > k; the sum may not be representable).
__device__ __forceinline__ bool length_fits(const Dims &D, int k, int len) { return len >= 0 && len <= D.max_seq - (k + 1); }

// grid = B sequences, block = 1024.  The target's choice after every node, merged from the LM head's partial maxima (one wave
// per row; the lowest token id wins a tie; without part_val it is in `that` already), then greedy acceptance by one thread, out
// of LDS: one launch, where a merge over the rows and a walk through global memory took two (4.8 + 4.8 us on chains, 6.4 + 5.3
// on trees of 13 nodes with 8016 partials a row).
//   chain: the longest draft prefix that the choices reproduce, and the bonus token
//   tree (the candidate tree the paper verifies, Sec. 3.1): from the root, step to the child whose token is the choice after the
//   current node (the lowest node index if several children carry it) until none does
__global__ __launch_bounds__(1024) void accept_kernel(StepIO io, const float *part_val, const int *part_idx, int n_part, int32_t *that)
{
    __shared__ int that_s[32], tok_s[32], par_s[32], path_s[32];   // k <= 31
    const int b = blockIdx.x, sq = io.k + 1, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, t = threadIdx.x;
    if (t < sq) {
        tok_s[t] = io.tokens[b * sq + t];
        if (io.parents) par_s[t] = io.parents[b * sq + t];
        if (!part_val) that_s[t] = that[b * sq + t];
        path_s[t] = -1;
    }
    if (part_val)
        for (int j = wave; j < sq; j += 16) {
            const size_t row = (size_t)(b * sq + j) * n_part;
            float bv = -INFINITY;
            int bi = 0x7FFFFFFF;
            constexpr int U = 8;
            for (int p0 = lane; p0 < n_part; p0 += U * 64) {
                float v[U];
                int id[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int p = p0 + u * 64;
                    v[u] = p < n_part ? part_val[row + p] : -INFINITY;
                    id[u] = p < n_part ? part_idx[row + p] : 0x7FFFFFFF;
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (v[u] > bv || (v[u] == bv && id[u] < bi)) { bv = v[u]; bi = id[u]; }
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const float ov = __shfl_xor(bv, off);
                const int oi = __shfl_xor(bi, off);
                if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            if (lane == 0) {
                if (bi == 0x7FFFFFFF) bi = 0;   // no logit of the row is a number
                that_s[j] = bi;
                that[b * sq + j] = bi;
            }
        }
    __syncthreads();
    if (t == 0) {
        int cur = 0, n = 0;
        path_s[0] = 0;
        for (;;) {
            int next = -1;
            if (!io.parents) {
                if (cur < io.k && tok_s[cur + 1] == that_s[cur]) next = cur + 1;
            } else {
                for (int c = cur + 1; c <= io.k; ++c)
                    if (par_s[c] == cur && tok_s[c] == that_s[cur]) { next = c; break; }
            }
            if (next < 0) break;
            cur = next;
            path_s[++n] = cur;
        }
        io.accepted_len[b] = n;
        io.next_token[b] = that_s[cur];
    }
    if (!io.parents) return;
    __syncthreads();
    if (t < sq) io.path[b * sq + t] = path_s[t];
}

// grid = (nkv, B, L), block = HD threads.  Moves the accepted rows to the front of the new ones, eight at a time: all of them are
// read before any is written.  Destinations lens + 1 .. lens + n never run ahead of the sources still to be read (path[i] >= i,
// increasing), so no eight disturb the next.  K rows in 16-byte records, eight rows per access of the workgroup (two bytes at a
// time an access took a cache line per eight threads); V, eight positions of one channel per record, an element per thread.
// 16 layers of 8 heads of 128, 32 sequences, 16 rows each: row after row, two bytes at a time 63 us a call, eight at a time 43.
template <int HD>
__global__ __launch_bounds__(HD) void kv_compact_kernel(Dims D, KvGeom kv, uint16_t *Kc, uint16_t *Vc, size_t kv_layer_elems, int k, const int32_t *lens,
                                                        const int32_t *accepted_len, const int32_t *path)
{
    constexpr int ROWS = 8, CPR = HD / 8;
    static_assert(HD == ROWS * CPR, "one record of K per thread");
    const int kvh = blockIdx.x, b = blockIdx.y, l = blockIdx.z, i = threadIdx.x;
    const int len = lens[b], n = accepted_len[b];
    if (!length_fits(D, k, len) || n < 0 || n > k) return;   // flagged by kv_commit_kernel
    if (!kv_pages_ok(kv, b, len, len + k)) return;                       // likewise: nothing moves through a bad page
    uint16_t *kc = Kc + (size_t)l * kv_layer_elems, *vc = Vc + (size_t)l * kv_layer_elems;
    path += b * (k + 1);
    int prev = 0;
    bool ok = true;
    for (int s0 = 1; ok && s0 <= n; s0 += ROWS) {
        int node[ROWS];      // of rows s0 ..; 0: not moved
#pragma unroll
        for (int u = 0; u < ROWS; ++u) node[u] = s0 + u <= n ? path[s0 + u] : 0;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            ok = ok && (s0 + u > n || (node[u] > prev && node[u] <= k));   // not an increasing path: leave the rest alone (flagged)
            if (ok && s0 + u <= n) prev = node[u];
            if (!ok || node[u] == s0 + u) node[u] = 0;
        }
        int mine = 0;        // of the row whose K record this thread moves
        u32x4 rec;
        uint16_t v[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            if (u == i / CPR) mine = node[u];
            if (node[u]) v[u] = vc[vcache_offset(kv, b, kvh, len + node[u], i)];
        }
        if (mine) rec = *reinterpret_cast<const u32x4 *>(kc + kcache_offset(kv, b, kvh, len + mine, i % CPR * 8));
        __syncthreads();     // another wave's rows may be this one's destinations
        if (mine) *reinterpret_cast<u32x4 *>(kc + kcache_offset(kv, b, kvh, len + s0 + i / CPR, i % CPR * 8)) = rec;
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
            if (node[u]) vc[vcache_offset(kv, b, kvh, len + s0 + u, i)] = v[u];
    }
}

// After kv_compact_kernel: lens[b] += accepted_len[b] + 1; malformed input raises the error flag
// and leaves lens[b] alone.
__global__ void kv_commit_kernel(Dims D, KvGeom kv, int B, int k, int32_t *lens, const int32_t *accepted_len, const int32_t *path,
                                 int32_t *err_flag)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int len = lens[b], n = accepted_len[b];
    bool ok = length_fits(D, k, len) && n >= 0 && n <= k;
    ok = ok && kv_pages_ok(kv, b, len, len + k);
    int prev = 0;
    for (int s = 1; ok && s <= n; ++s) {
        const int node = path[b * (k + 1) + s];
        ok = node > prev && node <= k;
        prev = node;
    }
    if (ok) lens[b] = len + n + 1;
    else *err_flag = 1;
}

__global__ void rollback_kernel(int B, int32_t *lens, const int32_t *accepted_len, const int32_t *new_lens)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    if (accepted_len) lens[b] += accepted_len[b] + 1;
    else lens[b] = new_lens[b];
}

// grid = (blocks of 32 positions that the rows touch, nkv), 256 threads.  ext layout [nkv][n_rows][HD]; Kc/Vc: the
// layer's pools.  One workgroup moves one (block, kv head): HD*64 bytes of K, whose 16-byte records are stored in another
// order, and as many of V, stored transposed (8 positions of one channel per record); both turn through LDS.  Everything in
// memory is read and written 16 bytes at a time, all loads of a thread in flight together: the kernel is bound by the
// copy rate (read + write) of the memory.  A pitch of HD + 8 elements keeps the 2-byte column accesses of a wave in
// separate banks (four rows 4 apart, 16 channels each).  4001 rows x 8 heads x 128, in or out: 17.4 -> 8.0 us (4.1 TB/s of reads and writes);
// 8192 rows 11.7 us (5.7 TB/s).
// The caller's rows are streamed (read or written once, here), the cache's are not: two layers of 8192 rows in and out 54.7 -> 47.0 us,
// eight of 4001 rows 121.5 -> 119.4 (sixteen calls of 7.3 from the host).  Rows that are not 16-byte aligned are read and written two bytes at
// a time on the caller's side only: 4001 rows x 8 heads x 128 in / out 17.5 / 19.1 us element by element, 7.2 / 7.4 so.
// A block that the rows cover only in part keeps its other rows: K rows and V elements outside are not written.
// Blocks that the table sends outside the pool are skipped (nothing written on either side) and raise the sticky flag.
template <int HD, bool IMPORT, bool ALIGNED>
__global__ __launch_bounds__(256) void kv_block_copy_kernel(KvGeom kv, uint16_t *Kc, uint16_t *Vc, int b, int t0, int n_rows, uint16_t *k_ext,
                                                            uint16_t *v_ext, int32_t *err_flag)
{
    constexpr int CPR = HD / 8, NREC = 32 * CPR, N = NREC / 256, PITCH = HD + 8;
    __shared__ __align__(16) uint16_t tile[32 * PITCH], ktile[32 * PITCH];
    const int blk = (t0 >> 5) + blockIdx.x, kvh = blockIdx.y;
    const int first = 32 * blk;                                   // position of the block's row 0
    if (!kv_pages_ok(kv, b, first, first)) {
        if (threadIdx.x == 0 && kvh == 0) *err_flag = 1;
        return;
    }
    const int lo = t0 > first ? t0 - first : 0, hi = min(32, t0 + n_rows - first);   // rows [lo, hi) of the block
    const size_t base = kv_block_offset(kv, kv_page(kv, b, blk), kvh);
    u32x4 *kc = reinterpret_cast<u32x4 *>(Kc + base), *vc = reinterpret_cast<u32x4 *>(Vc + base);
    // 16-byte records of the block's rows in the plain layout (row r, channels 8x..8x+7 at record r * CPR + x)
    const ptrdiff_t e0 = ((ptrdiff_t)kvh * n_rows + (first - t0)) * CPR;
    uint16_t *ke = k_ext + e0 * 8, *ve = v_ext + e0 * 8;
    auto get = [](const uint16_t *p) {
        if (ALIGNED) return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
        u32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = (uint32_t)p[2 * e] | ((uint32_t)p[2 * e + 1] << 16);
        return r;
    };
    auto put = [](uint16_t *p, const u32x4 &r) {
        if (ALIGNED) {
            __builtin_nontemporal_store(r, reinterpret_cast<u32x4 *>(p));
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = (uint16_t)(r[e >> 1] >> (16 * (e & 1)));
        }
    };
    // record rec of a K block: row, and which eight channels
    auto krow = [](int rec) { return rec / (CPR * 16) * 16 + (rec & 15); };
    auto kcol = [](int rec) { return rec / 64 % (CPR / 4) * 4 + (rec >> 4) % 4; };
    u32x4 k[N], v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int rec = threadIdx.x + 256 * i, row = rec / CPR;
        const bool in = row >= lo && row < hi;
        k[i] = v[i] = u32x4{0u, 0u, 0u, 0u};
        if (IMPORT) {
            if (in) {
                k[i] = get(ke + rec * 8);
                v[i] = get(ve + rec * 8);
            }
        } else {
            k[i] = kc[rec];
            v[i] = vc[rec];
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int rec = threadIdx.x + 256 * i;
        *reinterpret_cast<u32x4 *>(IMPORT ? &ktile[(rec / CPR) * PITCH + (rec % CPR) * 8] : &ktile[krow(rec) * PITCH + kcol(rec) * 8]) = k[i];
    }
    // record rec of a V block: channel (rec / 64) * 16 + rec % 16, positions 4q..4q+3 and 16+4q..16+4q+3, q = (rec / 16) % 4
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int rec = threadIdx.x + 256 * i;
        if (IMPORT) {
            *reinterpret_cast<u32x4 *>(&tile[(rec / CPR) * PITCH + (rec % CPR) * 8]) = v[i];
        } else {
            const int ch = (rec >> 6) * 16 + (rec & 15), q = (rec >> 4) & 3;
#pragma unroll
            for (int e = 0; e < 8; ++e) tile[(4 * q + (e & 3) + 16 * (e >> 2)) * PITCH + ch] = (uint16_t)(v[i][e >> 1] >> (16 * (e & 1)));
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int rec = threadIdx.x + 256 * i, row = IMPORT ? krow(rec) : rec / CPR, col = IMPORT ? kcol(rec) : rec % CPR;
        if (row < lo || row >= hi) continue;
        const u32x4 r = *reinterpret_cast<const u32x4 *>(&ktile[row * PITCH + col * 8]);
        if (IMPORT) kc[rec] = r;
        else put(ke + rec * 8, r);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int rec = threadIdx.x + 256 * i;
        if (!IMPORT) {
            const int row = rec / CPR;
            if (row >= lo && row < hi) put(ve + rec * 8, *reinterpret_cast<const u32x4 *>(&tile[row * PITCH + (rec % CPR) * 8]));
            continue;
        }
        const int ch = (rec >> 6) * 16 + (rec & 15), q = (rec >> 4) & 3;
        uint16_t x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = tile[(4 * q + (e & 3) + 16 * (e >> 2)) * PITCH + ch];
        if (lo == 0 && hi == 32) {
            u32x4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = (uint32_t)x[2 * e] | ((uint32_t)x[2 * e + 1] << 16);
            vc[rec] = r;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int row = 4 * q + (e & 3) + 16 * (e >> 2);
                if (row >= lo && row < hi) reinterpret_cast<uint16_t *>(vc + rec)[e] = x[e];
            }
        }
    }
}

// grid = M rows.  Plain fp32 -> packed bf16 hi/lo (no normalisation).
__global__ __launch_bounds__(256) void pack_act_kernel(const float *X, int K, int KT, uint16_t *A_hi, uint16_t *A_lo)
{
    const int m = blockIdx.x;
    for (int i = threadIdx.x; i < K; i += blockDim.x) {
        uint16_t hi, lo;
        split_bf16(X[(size_t)m * K + i], hi, lo);
        const size_t idx = packed_index(m, i, KT);
        A_hi[idx] = hi;
        A_lo[idx] = lo;
    }
}

// grid = M rows.  packed hi + lo -> fp32 [M][K].
__global__ __launch_bounds__(256) void unpack_act_kernel(const uint16_t *A_hi, const uint16_t *A_lo, int K, int KT, float *X)
{
    const int m = blockIdx.x;
    for (int i = threadIdx.x; i < K; i += blockDim.x) {
        const size_t idx = packed_index(m, i, KT);
        X[(size_t)m * K + i] = bf16_to_f32(A_hi[idx]) + bf16_to_f32(A_lo[idx]);
    }
}

// grid = (M, nq), block = d.  Already-rotated fp32 queries -> packed Q operand buffer.
__global__ void q_pack_kernel(Dims D, const float *q, int k, uint16_t *Qp, uint16_t *Qp_lo, int q_rows_pad)
{
    const int m = blockIdx.x, head = blockIdx.y, i = threadIdx.x;
    const int b = m / (k + 1), j = m % (k + 1);
    const int kvh = head / D.g, hl = head % D.g, r = j * D.g + hl;
    const size_t idx = ((size_t)b * D.nkv + kvh) * q_rows_pad * D.d + packed_index(r, i, D.d >> 5);
    uint16_t hi, lo;
    split_bf16(q[((size_t)m * D.nq + head) * D.d + i], hi, lo);
    Qp[idx] = hi;
    Qp_lo[idx] = lo;
}

// Rows that sequence b is ordered by: its length, if it fits.
__device__ __forceinline__ int length_or_zero(const Dims &D, int k, int len) { return length_fits(D, k, len) ? len : 0; }

// Turn of the sequence of the given rank among the lengths (0: the longest): the longer half in descending order, then the
// others in ascending order.  A compute unit takes its second workgroup half a launch after its first, so the longest meet the
// shortest.  Sequences in the order given / longest first / so, 8B shape, us of sssd_op_attention over cold caches: k = 4,
// B = 32, context 1024..4096 95 / 91 / 89, k = 8, B = 16, 1333..4000 64 / 61 / 61.
__device__ __forceinline__ int attention_turn(int rank, int B)
{
    const int first = (B + 1) / 2;
    return rank < first ? rank : B - 1 - (rank - first);
}

// Rank of sequence b among the lengths of a step (longest first, then by index); whole wave.
__device__ __forceinline__ int length_rank(const Dims &D, int B, int k, const int32_t *lens, int b, int lane)
{
    const int mine = length_or_zero(D, k, lens[b]);
    int rank = 0;
    for (int b0 = 0; b0 < B; b0 += 64) {
        const int o = b0 + lane, other = o < B ? length_or_zero(D, k, lens[o]) : -1;
        rank += __popcll(__ballot(other > mine || (other == mine && o < b)));
    }
    return rank;
}

// Validated lens and the row geometry of linear chains (kernel-level attention entry point).  grid = sequences, one wave.
__global__ void lens_kernel(Dims D, int B, int k, const int32_t *lens, int32_t *pos_base, AttnSeq *seq, int32_t *segments,
                            int32_t *rope_pos, uint32_t *anc, int32_t *err_flag, AttnPlan plan)
{
    const int b = blockIdx.x, lane = threadIdx.x;
    const int rank = length_rank(D, B, k, lens, b, lane);
    int len = lens[b];
    if (!length_fits(D, k, len)) {
        if (lane == 0) *err_flag = 1;
        len = 0;
    }
    if (lane == 0) {
        const AttnCut cut = attention_cut(plan, (len + k + 32) >> 5);
        pos_base[b] = len;
        seq[attention_turn(rank, B)] = AttnSeq{b, len, cut};
        segments[b] = cut.n;
    }
    if (lane <= k) {   // k <= 31
        rope_pos[b * (k + 1) + lane] = len + lane;
        anc[b * (k + 1) + lane] = 0xFFFFFFFFu >> (31 - lane);
    }
}

// Reorder a row-major bf16 matrix [N][K] into operand tiles (one 16-byte lane record per thread).
__global__ void pack_weight_kernel(const uint16_t *src, u32x4 *dst, int N, int K, int KT)
{
    const size_t rec = (size_t)blockIdx.x * blockDim.x + threadIdx.x;  // one 16-byte lane record
    const size_t total = (size_t)(N >> 4) * KT * 64;
    if (rec >= total) return;
    const int lane = (int)(rec & 63);
    const size_t tile = rec >> 6;
    const int kt = (int)(tile % KT);
    const int nt = (int)(tile / KT);
    const int n = nt * 16 + (lane & 15), k = kt * 32 + 8 * (lane >> 4);
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (k + 8 <= K) {
        v = *reinterpret_cast<const u32x4 *>(src + (size_t)n * K + k);
    } else if (k < K) {
        uint16_t tmp[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int e = 0; e < 8 && k + e < K; ++e) tmp[e] = src[(size_t)n * K + k + e];
        v = *reinterpret_cast<u32x4 *>(tmp);
    }
    dst[rec] = v;
}


// One sequence of a step, by one wave: validates its length and pages, leaves its cache row, cut and turn.
__device__ __forceinline__ void step_sequence(const Dims &D, const StepIO &io, const KvGeom &kv, const AttnPlan &plan, int b, int lane,
                                              int32_t *pos_base, AttnSeq *seq, int32_t *segments, int32_t *err_flag)
{
    const int rank = length_rank(D, io.B, io.k, io.lens, b, lane);
    const int len = io.lens[b];
    bool reject = !length_fits(D, io.k, len);   // the sequence must not write the cache: its rows would land on live data
    if (kv.table && !reject) {                  // every page the step reads or writes must lie in the pool
        bool bad = false;
        for (int blk = lane; blk <= (len + io.k) >> 5; blk += 64) {
            const int page = kv.table[(size_t)b * kv.blocks_per_seq + blk];
            bad = bad || page < 0 || page >= kv.n_pages;
        }
        reject = __any(bad);
    }
    if (lane != 0) return;
    // pos_base < 0 marks the rejected sequence for the K/V writers; readers take it as length 0
    pos_base[b] = reject ? -1 : len;
    const int rows = reject ? 0 : len;
    const AttnCut cut = attention_cut(plan, (rows + io.k + 32) >> 5);
    seq[attention_turn(rank, io.B)] = AttnSeq{b, rows, cut};
    segments[b] = cut.n;
    if (reject) *err_flag = 1;
}

// Geometry of row m of a step, by one wave: its depth and visible new rows, from the draft tree or the chain.
__device__ __forceinline__ void step_row(const Dims &D, const StepIO &io, int m, int lane, int32_t *rope_pos, uint32_t *anc, int32_t *err_flag)
{
    const int b = m / (io.k + 1), j = m % (io.k + 1), len = length_or_zero(D, io.k, io.lens[b]);
    int depth = j;
    uint32_t vis = 0xFFFFFFFFu >> (31 - j);
    if (io.parents) {
        // walk to the root over the parents that the lanes hold (through memory every node was a round trip); a parent outside
        // [0, node) is treated as node-1 and flagged
        const int mine = lane <= io.k ? io.parents[b * (io.k + 1) + lane] : 0;
        depth = 0;
        vis = 1u << j;
        for (int i = j; i > 0;) {
            int p = __builtin_amdgcn_readlane(mine, i);
            if (p < 0 || p >= i) {
                if (lane == 0) *err_flag = 1;
                p = i - 1;
            }
            i = p;
            vis |= 1u << i;
            ++depth;
        }
    }
    if (lane == 0) {
        rope_pos[m] = len + depth;
        anc[m] = vis;
    }
}

// grid = (row tiles of 16) * (chunks of EMBED_CHUNK channels) workgroups of 512 threads, and a wave for every row's geometry and every
// sequence beside them (in the rows' own waves the launch took 1 us longer).  Validates lens/tokens/parents; x = E[token]; packed
// x*gamma; sums of squares, one per row and chunk.
// What bounds it: the chain launch -> token -> row, and for many rows its stores (21 MB read and written at 512 x 4096 in 8.4 us).
// A wave takes a whole operand tile, so its records are 1 KiB in a row; with a row per workgroup each went to a line of its own, 16 bytes
// of 128.  Row per workgroup / chunks of 512 / of 256 channels, us: 512 rows of 4096 13.0 / 9.0 / 8.4, 160 rows 7.2 / 7.1 / 6.1, tree of
// 91 rows 7.8 / 6.9 / 6.7, 144 rows of 8192 8.7 / 8.0 / 8.0, 36 rows of 4096 5.4 / 5.2 / 5.2, five rows of 256 3.1 / 2.2 / 2.1.
__global__ __launch_bounds__(512) void fused_embed_kernel(Dims D, StepIO io, KvGeom kv, const uint16_t *embed, const uint16_t *gamma,
                                                          float *X, uint16_t *A_hi, uint16_t *A_lo, float *ssq,
                                                          int32_t *pos_base, AttnSeq *seq, int32_t *segments, int32_t *rope_pos,
                                                          uint32_t *anc, int32_t *err_flag, AttnPlan plan)
{
    constexpr int TILES = EMBED_CHUNK / 32 / 8;   // operand tiles per wave
    const int n_rows = io.B * (io.k + 1), chunks = embed_row_sums(D.h), tiles = (n_rows + 15) >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if ((int)blockIdx.x >= tiles * chunks) {
        const int of = ((int)blockIdx.x - tiles * chunks) * 8 + wave;
        if (of < io.B) step_sequence(D, io, kv, plan, of, lane, pos_base, seq, segments, err_flag);
        else if (of < io.B + n_rows) step_row(D, io, of - io.B, lane, rope_pos, anc, err_flag);
        return;
    }
    __shared__ float ss_s[8][16];
    const int tile = blockIdx.x / chunks, chunk = blockIdx.x % chunks, r = lane & 15, kg = lane >> 4;
    const int m = tile * 16 + r, KT = (D.h + 31) >> 5, kt0 = (chunk * 8 + wave) * TILES;
    const bool live = m < n_rows;
    int tok = io.tokens[live ? m : n_rows - 1];
    u32x4 g[TILES], e[TILES];   // the caller's arrays are only 2-byte aligned
#pragma unroll
    for (int t = 0; t < TILES; ++t) __builtin_memcpy(&g[t], gamma + min((kt0 + t) * 32 + kg * 8, D.h - 8), 16);
    if (tok < 0 || tok >= D.V) {
        if (live) *err_flag = 1;
        tok = 0;
    }
#pragma unroll
    for (int t = 0; t < TILES; ++t) __builtin_memcpy(&e[t], embed + (size_t)tok * D.h + min((kt0 + t) * 32 + kg * 8, D.h - 8), 16);
    float ss = 0.f;
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int col = (kt0 + t) * 32 + kg * 8;   // h is a multiple of 16
        f32x4 x[2];
        u32x4 hi, lo;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float x0 = __uint_as_float(e[t][c] << 16), x1 = __uint_as_float(e[t][c] & 0xFFFF0000u);
            uint32_t h2, l2;
            split_bf16x2(x0 * __uint_as_float(g[t][c] << 16), x1 * __uint_as_float(g[t][c] & 0xFFFF0000u), h2, l2);
            hi[c] = h2;
            lo[c] = l2;
            x[c >> 1][(c & 1) * 2] = x0;
            x[c >> 1][(c & 1) * 2 + 1] = x1;
            if (col < D.h) {
                ss += x0 * x0;
                ss += x1 * x1;
            }
        }
        if (live && col < D.h) {
            *reinterpret_cast<f32x4 *>(X + (size_t)m * D.h + col) = x[0];
            *reinterpret_cast<f32x4 *>(X + (size_t)m * D.h + col + 4) = x[1];
            const size_t idx = packed_index(m, col, KT);
            *reinterpret_cast<u32x4 *>(A_hi + idx) = hi;
            *reinterpret_cast<u32x4 *>(A_lo + idx) = lo;
        }
    }
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    if (kg == 0) ss_s[wave][r] = ss;
    __syncthreads();
    if (threadIdx.x < 16 && live) {
        float all = 0.f;
#pragma unroll
        for (int w = 0; w < 8; ++w) all += ss_s[w][threadIdx.x];
        ssq[(size_t)m * chunks + chunk] = all;
    }
}

// Plain read-only stream over a buffer: workgroup b reads the 16 KiB pieces b, b + grid, b + 2 grid, ...,
// each as four 16-byte loads per lane, all in flight together.  What it reaches is the read bandwidth a
// kernel on this device can get from HBM with no arithmetic in the way: the yardstick the weight
// streamers are held against.  (Measured on 2 GiB: 7.0-7.3 TB/s for 512 to 4096 workgroups of this shape;
// the same bytes fetched thread by thread at a grid-wide stride, four loads 8 MB apart per lane, reach
// 6.0 TB/s; 256 workgroups of 1024 threads with eight loads per lane, the launch shape of the weight
// streamers, 6.6-6.8 TB/s.)  The XOR of everything read goes to sink[workgroup] so that the loads are live.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4 *src, size_t n16, uint32_t *sink)
{
    constexpr size_t PIECE = 1024;   // records of a 16 KiB piece
    const size_t n_pieces = n16 / PIECE;
    u32x4 acc = u32x4{0u, 0u, 0u, 0u};
    for (size_t c = blockIdx.x; c < n_pieces; c += gridDim.x) {
        const u32x4 *p = src + c * PIECE + threadIdx.x;
        const u32x4 a = __builtin_nontemporal_load(p), b = __builtin_nontemporal_load(p + 256);
        const u32x4 cc = __builtin_nontemporal_load(p + 512), d = __builtin_nontemporal_load(p + 768);
        acc ^= a ^ b ^ cc ^ d;
    }
    for (size_t i = n_pieces * PIECE + (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256)
        acc ^= __builtin_nontemporal_load(src + i);
    uint32_t x = acc.x ^ acc.y ^ acc.z ^ acc.w;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x ^= __shfl_xor(x, off, 64);
    __shared__ uint32_t part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x == 0) sink[blockIdx.x] = part[0] ^ part[1] ^ part[2] ^ part[3];
}

__global__ __launch_bounds__(64) void die_check_kernel(uint64_t *found)
{
    const uint32_t die = own_die();
    if (threadIdx.x == 0) __hip_atomic_fetch_or(found, die > 7 ? (uint64_t)1 << 63 : (uint64_t)1 << ((die - blockIdx.x) & 7), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

hipError_t launch_die_check(uint64_t *found, hipStream_t s)
{
    hipLaunchKernelGGL(die_check_kernel, dim3(512), dim3(64), 0, s, found);
    return hipGetLastError();
}

hipError_t launch_stream_read(const void *src, size_t bytes, uint32_t *sink, int n_cu, hipStream_t s)
{
    const size_t n16 = bytes / 16;
    const int grid = n_cu * 2 < STREAM_READ_SINK_WORDS ? n_cu * 2 : STREAM_READ_SINK_WORDS;
    hipLaunchKernelGGL(stream_read_kernel, dim3(grid), dim3(256), 0, s, (const u32x4 *)src, n16, sink);
    return hipGetLastError();
}

hipError_t launch_accept(const StepIO &io, const float *part_val, const int *part_idx, int n_part, int32_t *that, hipStream_t s)
{
    hipLaunchKernelGGL(accept_kernel, dim3(io.B), dim3(1024), 0, s, io, part_val, part_idx, n_part, that);
    return hipGetLastError();
}

hipError_t launch_rollback(int B, int32_t *lens, const int32_t *accepted_len, const int32_t *new_lens, hipStream_t s)
{
    hipLaunchKernelGGL(rollback_kernel, dim3((B + 63) / 64), dim3(64), 0, s, B, lens, accepted_len, new_lens);
    return hipGetLastError();
}

hipError_t launch_kv_compact(const Dims &D, const KvGeom &kv, uint16_t *Kc, uint16_t *Vc, size_t kv_layer_elems, int B, int k,
                             int32_t *lens, const int32_t *accepted_len, const int32_t *path, int32_t *err_flag, hipStream_t s)
{
    const dim3 grid(D.nkv, B, D.L);
    if (D.d == 128) hipLaunchKernelGGL(kv_compact_kernel<128>, grid, dim3(128), 0, s, D, kv, Kc, Vc, kv_layer_elems, k, lens, accepted_len, path);
    else hipLaunchKernelGGL(kv_compact_kernel<64>, grid, dim3(64), 0, s, D, kv, Kc, Vc, kv_layer_elems, k, lens, accepted_len, path);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kv_commit_kernel, dim3((B + 63) / 64), dim3(64), 0, s, D, kv, B, k, lens, accepted_len, path, err_flag);
    return hipGetLastError();
}

hipError_t launch_kv_copy(const Dims &D, const KvGeom &kv, uint16_t *Kc_layer, uint16_t *Vc_layer, int b, int t0, int n_rows,
                          uint16_t *k_ext, uint16_t *v_ext, bool import, int32_t *err_flag, hipStream_t s)
{
    if (n_rows <= 0) return hipSuccess;
    const bool aligned = ((uintptr_t)k_ext | (uintptr_t)v_ext) % 16 == 0;   // rows are 128 or 256 bytes: every row is aligned then
    const dim3 grid(((t0 + n_rows - 1) >> 5) - (t0 >> 5) + 1, D.nkv);
#define SSSD_KVLAUNCH(HD, IN)                                                                                                              \
    do {                                                                                                                                   \
        if (aligned) hipLaunchKernelGGL((kv_block_copy_kernel<HD, IN, true>), grid, dim3(256), 0, s, kv, Kc_layer, Vc_layer, b, t0, n_rows, k_ext, v_ext, err_flag); \
        else hipLaunchKernelGGL((kv_block_copy_kernel<HD, IN, false>), grid, dim3(256), 0, s, kv, Kc_layer, Vc_layer, b, t0, n_rows, k_ext, v_ext, err_flag);        \
    } while (0)
    if (D.d == 128) {
        if (import) SSSD_KVLAUNCH(128, true);
        else SSSD_KVLAUNCH(128, false);
    } else {
        if (import) SSSD_KVLAUNCH(64, true);
        else SSSD_KVLAUNCH(64, false);
    }
#undef SSSD_KVLAUNCH
    return hipGetLastError();
}

hipError_t launch_pack_act(const float *X, int M, int K, uint16_t *A_hi, uint16_t *A_lo, hipStream_t s)
{
    hipLaunchKernelGGL(pack_act_kernel, dim3(M), dim3(256), 0, s, X, K, (K + 31) / 32, A_hi, A_lo);
    return hipGetLastError();
}

hipError_t launch_unpack_act(const uint16_t *A_hi, const uint16_t *A_lo, int M, int K, float *X, hipStream_t s)
{
    hipLaunchKernelGGL(unpack_act_kernel, dim3(M), dim3(256), 0, s, A_hi, A_lo, K, (K + 31) / 32, X);
    return hipGetLastError();
}

hipError_t launch_q_pack(const Dims &D, const float *q, int B, int k, uint16_t *Qp, uint16_t *Qp_lo, hipStream_t s)
{
    const int q_rows_pad = round_up(D.g * (D.max_k + 1), 16);
    hipLaunchKernelGGL(q_pack_kernel, dim3(B * (k + 1), D.nq), dim3(D.d), 0, s, D, q, k, Qp, Qp_lo, q_rows_pad);
    return hipGetLastError();
}

hipError_t launch_lens(const Dims &D, int B, int k, const int32_t *lens, int32_t *pos_base, AttnSeq *seq, int32_t *segments,
                       int32_t *rope_pos, uint32_t *anc, int32_t *err_flag, hipStream_t s)
{
    hipLaunchKernelGGL(lens_kernel, dim3(B), dim3(64), 0, s, D, B, k, lens, pos_base, seq, segments, rope_pos, anc, err_flag,
                       attention_plan(D, B, k));
    return hipGetLastError();
}

hipError_t launch_pack_weight(const uint16_t *src, uint16_t *dst, int N, int K, hipStream_t s)
{
    const int KT = (K + 31) / 32;
    const size_t total = (size_t)(N / 16) * KT * 64;
    const int threads = 256;
    const unsigned blocks = (unsigned)((total + threads - 1) / threads);
    hipLaunchKernelGGL(pack_weight_kernel, dim3(blocks), dim3(threads), 0, s, src, reinterpret_cast<u32x4 *>(dst), N, K, KT);
    return hipGetLastError();
}

hipError_t launch_fused_embed(const Dims &D, const StepIO &io, const KvGeom &kv, const uint16_t *embed, const uint16_t *gamma,
                              float *X, uint16_t *A_hi, uint16_t *A_lo, float *ssq, int32_t *pos_base, AttnSeq *seq, int32_t *segments, int32_t *rope_pos,
                              uint32_t *anc, int32_t *err_flag, hipStream_t s)
{
    const int n_rows = io.B * (io.k + 1), tiles = (n_rows + 15) / 16;
    hipLaunchKernelGGL(fused_embed_kernel, dim3(tiles * embed_row_sums(D.h) + (n_rows + io.B + 7) / 8), dim3(512), 0, s, D, io, kv, embed, gamma, X, A_hi, A_lo, ssq,
                       pos_base, seq, segments, rope_pos, anc, err_flag, attention_plan(D, io.B, io.k));
    return hipGetLastError();
}
