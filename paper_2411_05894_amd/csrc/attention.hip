// Causal grouped-query attention of the k+1 new rows against the per-sequence KV cache.
//
// Table 2 (App. B), attention row: A_out = softmax(Q K^T / sqrt(d) + M) V with
// K, V of shape (b, n_kv, s_kv + s_q, d).  Its FLOPs:IO ratio is ~ g*s_q, so the
// operation is bound by streaming the cache.  The mask M is never read as a tensor:
// every query row sees the old cache (rows below lens[b]) and, of the k+1 new rows, the
// ones named by a 32-bit word per query node -- itself and its ancestors in the draft
// tree (Sec. 3.1); for a linear chain that is "row j sees new rows 0..j".
//
// One workgroup owns one segment of one sequence's positions for one kv head.  A sequence is cut by
// its own length (attention_cut, by the kernel that validates the lens): caches with room to grow cost
// nothing, and what the other sequences hold changes no bit.  All g*(k+1) query rows that share the kv
// head are processed against the segment, up to four 16-row tiles at once, so every cached byte is read
// from HBM once per step (more tiles: the passes over the cache sit next to each other on a die and share
// its L2).
//
// The four waves of a workgroup take every fourth block of 32 positions each and carry ALL query rows
// through it: a block's K and V go from memory straight into the registers of the one wave that uses them
// (both pools are stored in operand order, 1 KiB in a row per load), nothing is staged through LDS and no
// wave waits for another until the segment is done.  As soon as a block's K (or V) has been used, the next
// block's is requested into the same registers.  The query operands, the same for every block, are read
// from LDS (one row tile: kept in registers).  Per block, wave and row tile:
//   S^T = K . Q^T        (A operand = 16 cached K rows)
//   online softmax in registers; the row statistics need only two cross-lane swaps
//   O^T += V^T . P^T     (A operand = V in its block-transposed cache order,
//                         B operand = the lane's own probabilities)
// The transposed forms are chosen so that the lane that owns a query row's
// statistics also owns that row's accumulator columns: no shuffles to rescale.
// At the end the waves bring their sums to one reference and add them up through LDS, each wave ending with a
// quarter of the channels.  A sequence that lies in one segment is finished by its workgroup itself; else the segments are merged in
// fixed order (deterministic): inside the launch where all segments of a (sequence, kv head) can run on one die (attention_in_die), by a
// second launch otherwise.  The second launch took 5.0-7.6 us and the gap in front of it; the workgroups of a die pass their sums on
// through its L2 and share the rows out: whole 8B step, one sequence of 2048 3421 -> 3357 us, four sequences of 32768, k = 8 2.6 us less a
// layer, sssd_op_attention of two sequences of 12345, k = 17 40.1 -> 38.1.
//
// What bounds it: the cache stream from a few MB per compute unit on (a compute unit pulls 24 GB/s with all of them at work, 537 MB in
// 87 us, and 32 GB/s beside idle ones, the longest of 32 ragged sequences, 2.1 MB in 66 us), below that the chain
// from the launch to the first operands and the final sums.  Measured against one wave per row tile with K and V staged
// through LDS behind two barriers per block, us of sssd_op_attention over cold caches (four small launches in it, 17 us):
// 8B shape B = 2, k = 17, context 12345 51 -> 45; B = 16, k = 31, 4000 132 -> 105; B = 32, k = 4, 1024..4096 90 -> 80; B = 4, k = 8,
// 32768 108 -> 105; 70B shape B = 16, k = 8, 2048 71 -> 60.  Two blocks ahead instead of one: 3-8 % slower at one and two row tiles (fewer
// registers are left to the second workgroup of a compute unit).  K rows in plain order: every load took half of sixteen cache lines, and
// streaming loads fetched some of them twice (B = 40, k = 3 69 us, 59 now).  Matrix and vector instructions in turn against the
// compiler's order, all probabilities first and then all products: B = 16, k = 31, 4000 104 -> 95, 70B shape B = 3, k = 15,
// 4000..12000 72 -> 65, 8B B = 2, k = 17 44.7 -> 42.6, one and two row tiles the same.
#include "kernels.h"

namespace {

__device__ __forceinline__ f32x4 mfma(const u32x4 &a, const u32x4 &b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

constexpr float NEG_BIG = -1.0e30f;
constexpr int MAX_TILES = 4;   // query-row tiles of a pass
constexpr int NWAVE = 4;       // waves of a workgroup, each on every fourth block of the segment

// max / sum over the four lanes 16 apart that share a query row
__device__ __forceinline__ float rows_max(float x)
{
    auto h = __builtin_amdgcn_permlane32_swap(f32_bits(x), f32_bits(x), false, false);
    x = fmaxf(bits_f32(h[0]), bits_f32(h[1]));
    h = __builtin_amdgcn_permlane16_swap(f32_bits(x), f32_bits(x), false, false);
    return fmaxf(bits_f32(h[0]), bits_f32(h[1]));
}
__device__ __forceinline__ float rows_sum(float x)
{
    auto h = __builtin_amdgcn_permlane32_swap(f32_bits(x), f32_bits(x), false, false);
    x = bits_f32(h[0]) + bits_f32(h[1]);
    h = __builtin_amdgcn_permlane16_swap(f32_bits(x), f32_bits(x), false, false);
    return bits_f32(h[0]) + bits_f32(h[1]);
}

__device__ __forceinline__ float wave_max(float x)   // in every lane, without LDS
{
    x = fmaxf(x, bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x128, 0xF, 0xF, true)));   // rotated by 8, 4, 2, 1 lanes of 16
    x = fmaxf(x, bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x124, 0xF, 0xF, true)));
    x = fmaxf(x, bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x122, 0xF, 0xF, true)));
    x = fmaxf(x, bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x121, 0xF, 0xF, true)));
    return rows_max(x);
}

// The segments of ROWS query rows r0, r0 + step, ... (below r_end) of (sequence b, kv head kvh) merged by one wave, in fixed order.  The
// wave reads the rows' partial outputs of 4*U segments in one round of independent loads: lanes 16s..16s+15 take segment s, s+4, ...
// with 8 channels each; then the four lane groups are summed, each ending with two of the eight.  MANY: more than 4*U segments, in
// rounds.  DIE: workgroups of this launch, on this die, stored them.
template <int HD, int ROWS, int U, bool MANY, bool DIE>
__device__ __forceinline__ void merge_rows(const Dims &D, const AttnArgs &a, int q_rows_pad, int b, int kvh, int r0, int step, int r_end, int n_splits, int lane)
{
#pragma clang fp contract(off)   // a row's bits must not depend on how many are merged at once: fused where it says so
    constexpr int LPR = HD / 8;   // lanes that cover a row of HD channels, 8 each
    const int KTq = (D.qd + 31) >> 5;
    const int sg = lane >> 4, cl = lane & 15;
    const size_t slot0 = ((size_t)kvh * a.B + b) * a.plan.share;
    const float *part_o = a.part_o + slot0 * q_rows_pad * HD, *part_ml = a.part_ml + slot0 * q_rows_pad * 2;
    const DieBuffer die_o(part_o, (size_t)n_splits * q_rows_pad * HD * sizeof(float)), die_ml(part_ml, (size_t)n_splits * q_rows_pad * sizeof(float2));
    auto stats = [&](int segment, int r) {
        const int at = segment * q_rows_pad + r;
        return DIE ? die_ml.load2(at * 8) : *reinterpret_cast<const float2 *>(part_ml + (size_t)at * 2);
    };
    auto row = [&](int i) { return min(r0 + i * step, r_end - 1); };

    float num[ROWS][8], den[ROWS], m_star[ROWS];
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        m_star[i] = MANY ? stats(min(lane, n_splits - 1), row(i)).x : 0.f;   // at most ATTN_MAX_SEGMENTS, a lane each
        den[i] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) num[i][e] = 0.f;
    }
    for (int base = 0; base < (MANY ? n_splits : 1); base += 4 * U) {
        f32x4 pv[ROWS][U][2];
        float2 ml[ROWS][U];
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) {   // past the last segment: that one again, not added
                const int s = min(base + 4 * u + sg, n_splits - 1), at = (s * q_rows_pad + row(i)) * HD + min(cl, LPR - 1) * 8;
                ml[i][u] = stats(s, row(i));
                if (DIE) {
                    pv[i][u][0] = die_o.load4(at * 4);
                    pv[i][u][1] = die_o.load4(at * 4, 16);
                } else {
                    pv[i][u][0] = *reinterpret_cast<const f32x4 *>(part_o + at);
                    pv[i][u][1] = *reinterpret_cast<const f32x4 *>(part_o + at + 4);
                }
            }
        if (base == 0) {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                if (MANY) {
                    m_star[i] = wave_max(m_star[i]);
                } else {
                    float m = ml[i][0].x;
#pragma unroll
                    for (int u = 1; u < U; ++u) m = fmaxf(m, ml[i][u].x);
                    m_star[i] = rows_max(m);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool on = base + 4 * u + sg < n_splits;
                const float w = __builtin_amdgcn_exp2f(ml[i][u].x - m_star[i]);
                den[i] = on ? __builtin_fmaf(w, ml[i][u].y, den[i]) : den[i];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    num[i][e] = on ? __builtin_fmaf(w, pv[i][u][0][e], num[i][e]) : num[i][e];
                    num[i][4 + e] = on ? __builtin_fmaf(w, pv[i][u][1][e], num[i][4 + e]) : num[i][4 + e];
                }
            }
    }
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
        const float inv = 1.f / rows_sum(den[i]);
        float half[4], two[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) {   // lane groups 0 and 1 keep channels 0..3, 2 and 3 channels 4..7
            const auto h = __builtin_amdgcn_permlane32_swap(f32_bits(num[i][e]), f32_bits(num[i][4 + e]), false, false);
            half[e] = bits_f32(h[0]) + bits_f32(h[1]);
        }
#pragma unroll
        for (int e = 0; e < 2; ++e) {   // groups 0 and 2 the first two of them
            const auto h = __builtin_amdgcn_permlane16_swap(f32_bits(half[e]), f32_bits(half[2 + e]), false, false);
            two[e] = bits_f32(h[0]) + bits_f32(h[1]);
        }
        const int r = r0 + i * step;
        if (r < r_end && cl < LPR) {
            uint32_t hi, lo;
            split_bf16x2(two[0] * inv, two[1] * inv, hi, lo);
            const int j = a.by_g(r), hl = r - j * D.g, m = b * (a.k + 1) + j;
            const size_t idx = packed_index(m, (kvh * D.g + hl) * HD + cl * 8 + (sg >> 1) * 4 + (sg & 1) * 2, KTq);
            *reinterpret_cast<uint32_t *>(a.out_hi + idx) = hi;
            *reinterpret_cast<uint32_t *>(a.out_lo + idx) = lo;
        }
    }
}

// grid = B * share * kv heads * passes over the row tiles; block = four waves; RT row tiles per pass; ONCE: a single pass.
// Workgroups 8 apart run on one die, where the passes and then the heads of a segment follow each other: they read one page
// (64 KiB of K at eight heads of 128) at about the same time.  Two waves per SIMD: two workgroups fit a compute unit.
template <int HD, int RT, bool ONCE>
__global__ __launch_bounds__(NWAVE * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_partial_kernel(Dims D, AttnArgs a, int q_rows_pad)
{
    constexpr int KS = HD / 32, DT = HD / 16;
    constexpr int NREC = 4 * HD;             // 16-byte records of a block of 32 positions, K and V alike
    constexpr bool QREG = RT == 1;           // query operands in registers, else in LDS
    constexpr int QAHEAD = RT == 4 ? 1 : 3;  // pairs of them fetched ahead: four tiles leave registers for one
    constexpr int QREC = QREG ? 0 : RT * KS * 2 * 64, RRED = NWAVE * (NWAVE - 1) * (RT <= 3 ? RT : 2) * (DT / 4) * 64;   // records of the query tiles, of the final sums
    __shared__ u32x4 lds[QREC > RRED ? QREC : RRED];
    __shared__ float2 ml_s[NWAVE][RT * 16];
    __shared__ int way_s;
    __shared__ uint32_t vis_s[RT * 16];      // visible new rows of every query row: bit i = cache row len + i

    int pass = 0, turn, kvh, segment;
    const int passes = a.plan.passes, share = a.plan.share;
    {
        int id = blockIdx.x;
        if (a.hand.words) {   // all segments of a (sequence, kv head) on one die, its passes next to each other
            // Heads of one sequence and, by turn, of different sequences on a die: with one head per die each die would read the same
            // eighth of every page.
            const int slot = id >> 3, x = a.by_passes(slot), row = a.by_share(x), u = row * 8 + ((id - row) & 7);
            pass = slot - x * passes;
            segment = x - row * share;
            turn = a.by_nkv(u);
            kvh = u - turn * D.nkv;
        } else {
            if (passes > 1) {
                const int n = a.B * share * D.nkv, sets = n & ~7;
                if (id < sets * passes) {
                    const int x = a.by_passes(id >> 3);
                    pass = (id >> 3) - x * passes;
                    id = x * 8 + (id & 7);
                } else {
                    const int r = id - sets * passes;
                    pass = r / (n - sets);
                    id = sets + r % (n - sets);
                }
            }
            const int whole = (a.B * share) & ~7;
            int wg;   // (turn, segment)
            if (id < whole * D.nkv) {
                const int x = a.by_nkv(id >> 3);
                wg = x * 8 + (id & 7);
                kvh = (id >> 3) - x * D.nkv;
            } else {
                const int r = id - whole * D.nkv, x = a.by_nkv(r);
                wg = whole + x;
                kvh = r - x * D.nkv;
            }
            turn = a.by_share(wg);
            segment = wg - turn * share;
        }
    }
    const AttnSeq me = a.seq[turn];
    const int b = me.b, len = me.len, total = len + a.k + 1;   // a rejected sequence is read as empty
    const AttnCut cut = me.cut;
    if (segment >= cut.n) return;
    const int first_blk = segment * cut.each, n_blk = min(cut.each, ((total + 31) >> 5) - first_blk);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int q = lane >> 4, c = lane & 15;
    const int rt0 = pass * RT, n_it = n_blk > wave ? (n_blk - wave + NWAVE - 1) / NWAVE : 0;

    // Pages of this wave's blocks: lane l keeps the page of its block number 64 * chunk + l, one chunk ahead of the next.
    auto load_pages = [&](int chunk) { return kv_page(a.kv, b, min(first_blk + wave + NWAVE * (64 * chunk + lane), a.kv.blocks_per_seq - 1)); };
    int chunk = 0, pg = load_pages(0), pg_next = load_pages(1);

    // Query operands of tile t: hi and lo parts (q ~= hi + lo, so the scores carry fp32-level accuracy although K is bf16)
    auto query = [&](int t, int ks, int part) {
        const int rt = min(rt0 + t, (q_rows_pad >> 4) - 1);   // the last pass may have tiles to spare: they repeat one
        const uint16_t *base = part ? a.Qp_lo : a.Qp;
        return reinterpret_cast<const u32x4 *>(base + ((size_t)b * D.nkv + kvh) * q_rows_pad * HD) + ((size_t)rt * KS + ks) * 64;
    };
    u32x4 qreg[QREG ? KS : 1][2];
    constexpr int QPT = QREG ? 1 : RT * KS * 2 / NWAVE;   // operand tiles copied per wave
    u32x4 qcopy[QPT];
    if (QREG) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            qreg[QREG ? ks : 0][0] = query(0, ks, 0)[lane];
            qreg[QREG ? ks : 0][1] = query(0, ks, 1)[lane];
        }
    } else {
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int x = wave * QPT + i;   // [tile][ks][part]
            qcopy[i] = query(x / (2 * KS), (x >> 1) % KS, x & 1)[lane];
        }
    }

    // A block's operands.  Every load is issued unconditionally, because a load under a branch would make every later wait a full drain;
    // past the wave's last block the buffer they read has no records and the loads return at once without one.  (Reading the last block
    // again instead kept the final sums waiting for memory: 2 us of a segment's time.)  A single pass streams; several passes find K, and
    // mostly V, in the die's L2.
    u32x4 k[2][KS], v[DT];
    auto block = [&](const uint16_t *pool, int i) {   // the wave's block i
        const int at = i < n_it ? i : 0;
        const int x = __builtin_amdgcn_readlane(at >> 6 == chunk ? pg : pg_next, at & 63);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<u32x4 *>(reinterpret_cast<const u32x4 *>(pool) + ((size_t)x * D.nkv + kvh) * NREC), 0,
                                                 i < n_it ? NREC * 16 : 0, 0x00027000);
    };
    constexpr int STREAM = 2;   // non-temporal
    auto load_k = [&](int i) {
        const auto p = block(a.Kc, i);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                k[u][ks] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(p, lane * 16, (u * KS + ks) * 1024, ONCE ? STREAM : 0));
    };
    auto load_v = [&](int i) {
        const auto p = block(a.Vc, i);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) v[dt] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(p, lane * 16, dt * 1024, STREAM));
    };
    const bool has_new = (first_blk + n_blk) * 32 > len;   // the segment holds new rows
    auto visible = [&](int row) { return a.anc[b * (a.k + 1) + min(a.by_g(rt0 * 16 + row), a.k)]; };   // query row -> node of the chain or tree
    constexpr bool VREG = RT <= 3;   // in registers, else in LDS
    uint32_t vis[VREG ? RT : 1];
#pragma unroll
    for (int t = 0; t < (VREG ? RT : 1); ++t) vis[t] = 0;
    if (has_new) {
        if (VREG) {
#pragma unroll
            for (int t = 0; t < (VREG ? RT : 1); ++t) vis[t] = visible(t * 16 + c);
        } else if ((int)threadIdx.x < RT * 16) {
            vis[0] = visible(threadIdx.x);
        }
    }
    load_k(0);
    load_v(0);
    // One row tile has no other scheduling barriers: without these the compiler moves loads of the first block (which it takes out of the
    // loop) behind products, and their latencies add up (16 rows of four heads of 128, 200 positions: 7.2 us, 5.7 with them).
    if (QREG) __builtin_amdgcn_sched_barrier(0);

    f32x4 o[RT][DT];
    float m_run[RT], l_run[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        m_run[t] = NEG_BIG;
        l_run[t] = 0.f;
    }
    if (!QREG) {
#pragma unroll
        for (int i = 0; i < QPT; ++i) lds[(wave * QPT + i) * 64 + lane] = qcopy[i];
    }
    if (!VREG && threadIdx.x < RT * 16) vis_s[threadIdx.x] = vis[0];
    if (!QREG) __syncthreads();
    const float scale = 1.4426950408889634f * rsqrtf((float)HD);  // log2(e)/sqrt(d)

    // A block: scores of every tile, their maxima, then probabilities and results.  A wave issues in order, and alone on its SIMD it
    // keeps matrix and vector units busy only if their instructions alternate: the maxima of a tile are taken between the score
    // MFMAs of the next, the probabilities of a tile between the result MFMAs of the one before.
    for (int i = 0; i < n_it; ++i) {
        if (i >> 6 != chunk) {   // once per 64 blocks
            chunk = i >> 6;
            pg = pg_next;
            pg_next = load_pages(chunk + 1);
        }
        const int t0 = (first_blk + wave + NWAVE * i) * 32;
        int ql = lane;
        asm volatile("" : "+v"(ql));   // the query operands are read again for every block: hoisted, they would not fit the registers
        f32x4 s[RT][2];                // s[t][u][r]: score of position t0 + 16u + 4q + r for query row c of tile t
        float mx[RT];
        bool grow = false;
        u32x4 qx[QREG ? 1 : QAHEAD][2];
        auto fetch_q = [&](int x) {
            qx[x % QAHEAD][0] = lds[x * 128 + ql];
            qx[x % QAHEAD][1] = lds[x * 128 + 64 + ql];
        };
        auto maxima = [&](int t, int part) {   // in four parts
            if (part == 0) mx[t] = fmaxf(fmaxf(fmaxf(s[t][0][0], s[t][0][1]), s[t][0][2]), s[t][0][3]);
            if (part == 1) mx[t] = fmaxf(fmaxf(fmaxf(fmaxf(mx[t], s[t][1][0]), s[t][1][1]), s[t][1][2]), s[t][1][3]);
            if (part == 2) mx[t] = rows_max(mx[t]);
            if (part == 3) {
                mx[t] *= scale;
                grow = grow || mx[t] > m_run[t] + 8.f;
            }
        };
        if (!QREG) {
#pragma unroll
            for (int x = 0; x < QAHEAD; ++x) fetch_q(x);
        }
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            s[t][0] = s[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int x = t * KS + ks;
                const u32x4 hi = QREG ? qreg[QREG ? ks : 0][0] : qx[x % QAHEAD][0], lo = QREG ? qreg[QREG ? ks : 0][1] : qx[x % QAHEAD][1];
#pragma unroll
                for (int u = 0; u < 2; ++u) s[t][u] = mfma(k[u][ks], hi, s[t][u]);
#pragma unroll
                for (int u = 0; u < 2; ++u) s[t][u] = mfma(k[u][ks], lo, s[t][u]);
                if (!QREG && x + QAHEAD < RT * KS) fetch_q(x + QAHEAD);
                if (t > 0) {
#pragma unroll
                    for (int part = ks * 4 / KS; part < (ks + 1) * 4 / KS; ++part) maxima(t - 1, part);
                }
                if (!QREG) __builtin_amdgcn_sched_barrier(0);
            }
            if (t0 + 32 > len) {   // the block holds new rows: apply the nodes' visibility words
                const uint32_t seen = VREG ? vis[VREG ? t : 0] : vis_s[t * 16 + c];
                const int at = t0 - len;   // bit p of `in`: position p of the block is visible; old cache always is
                const uint32_t in = at > 31 ? 0u : (at >= 0 ? seen >> at : seen << -at | ((1u << -at) - 1u)), mine = in >> (4 * q);
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (!(mine & (1u << (16 * u + r)))) s[t][u][r] = -INFINITY;
            }
        }
        load_k(i + 1);
        if (QREG) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int part = 0; part < 4; ++part) maxima(RT - 1, part);
        // The exponent's reference m_run follows the running maximum lazily: it moves (and the accumulators are rescaled)
        // only when some row's maximum has outgrown it by more than 2^8, so most blocks skip the rescale.  Any reference gives
        // the same softmax; probabilities stay below 2^8 and the partial (o, l, m_run) handed on is consistent with it.
        if (__any(grow)) {
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const float m_new = mx[t] > m_run[t] + 8.f ? mx[t] : m_run[t], alpha = __builtin_amdgcn_exp2f(m_run[t] - m_new);
                m_run[t] = m_new;
                if (i == 0) continue;   // nothing to rescale yet
                l_run[t] *= alpha;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) o[t][dt] *= alpha;
            }
        }
        // p ~= hi + lo: the probabilities keep ~16 mantissa bits.  Two of a tile's eight per call, in four parts.
        uint32_t pk[2][4], pkl[2][4];
        float p0, p1;
        auto probs = [&](int t, int e, int part) {
            uint32_t &hi = pk[t & 1][e], &lo = pkl[t & 1][e];
            if (part == 0) {
                p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][e >> 1][2 * (e & 1)], scale, -m_run[t]));
                p1 = __builtin_fmaf(s[t][e >> 1][2 * (e & 1) + 1], scale, -m_run[t]);
            }
            if (part == 1) {
                p1 = __builtin_amdgcn_exp2f(p1);
                l_run[t] += p0;
            }
            if (part == 2) {
                hi = pack_bf16x2(p0, p1);
                l_run[t] += p1;
                p0 -= bits_f32(hi << 16);
            }
            if (part == 3) lo = pack_bf16x2(p0, p1 - bits_f32(hi & 0xFFFF0000u));
        };
#pragma unroll
        for (int x = 0; x < 16; ++x) probs(0, x >> 2, x & 3);
        if (RT > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            const u32x4 pb = u32x4{pk[t & 1][0], pk[t & 1][1], pk[t & 1][2], pk[t & 1][3]}, pl = u32x4{pkl[t & 1][0], pkl[t & 1][1], pkl[t & 1][2], pkl[t & 1][3]};
#pragma unroll
            for (int x = 0; x < 2 * DT; ++x) {   // hi and lo of two tiles of channels in turn
                const int dt = x >> 2 << 1 | (x & 1);
                o[t][dt] = mfma(v[dt], x & 2 ? pl : pb, o[t][dt]);
                if (t + 1 < RT) {
#pragma unroll
                    for (int y = x * 16 / (2 * DT); y < (x + 1) * 16 / (2 * DT); ++y) probs(t + 1, y >> 2, y & 3);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        load_v(i + 1);
    }

    // The waves' sums added up, on one reference per query row: every wave ends with a quarter of the channels of all rows.  It stores
    // the other three quarters as they are; who takes them has all four references and weighs them while adding.  One wave per SIMD
    // issues an instruction every four cycles: in two halving steps, selected by wave and scaled first, three tiles took 3.0 us of
    // which these take 1.9.
    constexpr int QT = DT / 4, TR = RT <= 3 ? RT : 2;   // channel tiles of a quarter; row tiles exchanged at a time
    f32x4 *red = reinterpret_cast<f32x4 *>(lds);
    const int dt0 = wave * QT;
    f32x4 own[RT][QT];
    if (RT > 1) __syncthreads();   // the query tiles have been read
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        l_run[t] = rows_sum(l_run[t]);
        if (q == 0) ml_s[wave][t * 16 + c] = float2{m_run[t], l_run[t]};
    }
#pragma unroll
    for (int w = 0; w < NWAVE; ++w)
        if (w == wave)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int x = 0; x < QT; ++x) own[t][x] = o[t][w * QT + x];
    auto part = [&](int quarter, int from, int t, int x) -> f32x4 & {   // of wave `from`, for the wave of `quarter`
        return red[(((quarter * (NWAVE - 1) + from - (from > quarter ? 1 : 0)) * TR + t % TR) * QT + x) * 64 + lane];
    };
    auto give = [&](int t0) {
#pragma unroll
        for (int w = 0; w < NWAVE; ++w)
            if (w != wave)
#pragma unroll
                for (int t = t0; t < t0 + TR; ++t)
#pragma unroll
                    for (int x = 0; x < QT; ++x) part(w, wave, t, x) = o[t][w * QT + x];
    };
    // What the others left for this wave, all of it requested before any is used; index i: wave + i, so in an order that the quarter fixes.
    f32x4 taken[TR][NWAVE][QT];
    float2 st[TR][NWAVE];
    auto take = [&](int t0) {
#pragma unroll
        for (int i = 0; i < NWAVE; ++i) {
            const int w = (wave + i) & (NWAVE - 1);
#pragma unroll
            for (int t = 0; t < TR; ++t) {
                st[t][i] = ml_s[w][(t0 + t) * 16 + c];
                if (i > 0)
#pragma unroll
                    for (int x = 0; x < QT; ++x) taken[t][i][x] = part(wave, w, t0 + t, x);
            }
        }
    };
    give(0);
    __syncthreads();
    take(0);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        if (t > 0 && t % TR == 0) {
            __syncthreads();
            give(t);
            __syncthreads();
            take(t);
        }
        const float2 (&s4)[NWAVE] = st[t % TR];
        const float m_all = fmaxf(fmaxf(s4[0].x, s4[1].x), fmaxf(s4[2].x, s4[3].x));
        float l_all = 0.f;
        f32x4 y[QT];   // y[x][r]: channel (dt0 + x) * 16 + 4q + r of query row c of tile t
#pragma unroll
        for (int i = 0; i < NWAVE; ++i) {
            const float f = __builtin_amdgcn_exp2f(s4[i].x - m_all);
            l_all += s4[i].y * f;
#pragma unroll
            for (int x = 0; x < QT; ++x) y[x] = i ? y[x] + taken[t % TR][i][x] * f : own[t][x] * f;
        }
        const int row = (rt0 + t) * 16 + c;
        if (rt0 + t >= a.row_tiles) continue;
        if (cut.n == 1) {   // the whole sequence: the packed operands of the O projection
            const int jj = a.by_g(row), hl = row - jj * D.g;
            if (jj <= a.k) {
                const float inv = 1.f / l_all;
                const int m = b * (a.k + 1) + jj, KTq = (D.qd + 31) >> 5;
                const size_t idx = packed_index(m, (kvh * D.g + hl) * HD + 4 * q, KTq);
#pragma unroll
                for (int x = 0; x < QT; ++x) {
                    const int dt = dt0 + x;
                    uint32_t h0, l0, h1, l1;
                    split_bf16x2(y[x][0] * inv, y[x][1] * inv, h0, l0);
                    split_bf16x2(y[x][2] * inv, y[x][3] * inv, h1, l1);
                    // channels dt*16 + 4q ..+3: half of lane record 2*(dt%2) + q/2 of k-tile dt/2 of the head
                    const size_t at = idx + (size_t)(dt >> 1) * 512 + (size_t)(dt & 1) * 256;
                    *reinterpret_cast<uint2 *>(a.out_hi + at) = uint2{h0, h1};
                    *reinterpret_cast<uint2 *>(a.out_lo + at) = uint2{l0, l1};
                }
            }
        } else {
            const size_t at = (((size_t)kvh * a.B + b) * a.plan.share + segment) * q_rows_pad + row;
            float *po = a.part_o + at * HD;
#pragma unroll
            for (int x = 0; x < QT; ++x) *reinterpret_cast<f32x4 *>(po + (dt0 + x) * 16 + 4 * q) = y[x];
            if (wave == 0 && q == 0) *reinterpret_cast<float2 *>(a.part_ml + at * 2) = float2{m_all, l_all};
        }
    }
    if (cut.n == 1 || !a.hand.words) return;
    const int group = (turn * D.nkv + kvh) * passes + pass;   // by turn, not by sequence: both count to B
    HandWay way = hand_wait(a.hand, group, cut.n, hand_arrive(a.hand, group), &way_s);
    if (way == HAND_TURN_IN) way = hand_turn_in(a.hand, group, cut.n, &way_s);
    uint64_t left = way == HAND_SHARE ? hand_leave(a.hand, group) : 0;   // under way while the shares are done
    if (way != HAND_NOTHING) {   // the rows of this pass shared out over the waves of all segments
        const int r_end = min(D.g * (a.k + 1), (rt0 + RT) * 16), step = (way == HAND_ALL ? 1 : cut.n) * NWAVE;
        int r = rt0 * 16 + (way == HAND_ALL ? wave : wave * cut.n + segment);
        // as many rows at once as the wave has, up to four, when they have few segments
#define SSSD_MERGE(ROWS, U, MANY) for (; r < r_end; r += ROWS * step) merge_rows<HD, ROWS, U, MANY, true>(D, a, q_rows_pad, b, kvh, r, step, r_end, cut.n, lane)
        if (cut.n > 8) SSSD_MERGE(1, 5, true);
        else if (cut.n > 4) {
            if (r + step < r_end) SSSD_MERGE(2, 2, false);
            else SSSD_MERGE(1, 2, false);
        } else {
            if (r + 2 * step < r_end) SSSD_MERGE(4, 1, false);
            else if (r + step < r_end) SSSD_MERGE(2, 1, false);
            else SSSD_MERGE(1, 1, false);
        }
#undef SSSD_MERGE
    }
    if (way != HAND_SHARE) left = hand_leave(a.hand, group);
    hand_clear(a.hand, group, cut.n, left);
}

// The merge as a launch of its own: one wave per (sequence, kv head, query row), 4 waves per block.
template <int HD>
__global__ __launch_bounds__(256) void attn_combine_kernel(Dims D, AttnArgs a, int q_rows_pad)
{
    const int R = D.g * (a.k + 1);
    const int task = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (task >= a.B * D.nkv * R) return;
    const int r = task % R, kvh = (task / R) % D.nkv, b = task / (R * D.nkv);
    const int n_splits = a.segments[b];    // at most ATTN_MAX_SEGMENTS
    if (n_splits == 1) return;             // finished by its workgroup
    // nine at a time cost registers: B = 12, k = 31, context 900..2700 81 us of attention, five 78
    merge_rows<HD, 1, 5, true, false>(D, a, q_rows_pad, b, kvh, r, 1, r + 1, n_splits, threadIdx.x & 63);
}

template <int HD> hipError_t launch_partial(const Dims &D, const AttnArgs &a, int q_rows_pad, hipStream_t s)
{
    const int passes = a.plan.passes, rt = (a.row_tiles + passes - 1) / passes;
    const dim3 grid(a.B * a.plan.share * D.nkv * passes);
#define SSSD_ALAUNCH(RT, ONCE) hipLaunchKernelGGL((attn_partial_kernel<HD, RT, ONCE>), grid, dim3(NWAVE * 64), 0, s, D, a, q_rows_pad)
    switch (rt) {
    case 1: SSSD_ALAUNCH(1, true); break;
    case 2: if (passes == 1) SSSD_ALAUNCH(2, true); else SSSD_ALAUNCH(2, false); break;
    case 3: if (passes == 1) SSSD_ALAUNCH(3, true); else SSSD_ALAUNCH(3, false); break;
    default: if (passes == 1) SSSD_ALAUNCH(4, true); else SSSD_ALAUNCH(4, false); break;
    }
#undef SSSD_ALAUNCH
    return hipGetLastError();
}

}  // namespace

// Passes over the cache for `tiles` row tiles, heads = sequences x kv heads: as few as MAX_TILES allows; for four tiles, and for ten to
// fifteen, one more (two of two; passes of three) or two more (ten tiles: of two) where that gives one workgroup to every compute unit or
// to at least three quarters of them, and one more where the fewest leave a second round to few workgroups.  A workgroup's query tiles,
// first operands and final sums grow with its tiles, and are most of its time when a wave has only a block or two; the passes share the
// cache's bytes in the die's L2.  More passes than that cost 2-7 % at 20000 positions.  sssd_op_attention over cold caches, us, fewest / more
// (workgroups for one segment), contexts 150, 500, 2048, 8000:
//   four tiles, 8B, k = 15: B = 1 (8 / 16) 23.6 / 19.4, 25.1 / 22.3, 26.9 / 24.4, 32.2 / 27.3; B = 8 (64 / 128) 29.7 / 24.0, 34.6 / 30.3, 40.1 / 37.1,
//     69.8 / 70.0; B = 14 (112 / 224) 31.6 / 25.8, 38.7 / 27.6, 51.4 / 43.6, 99.6 / 92.7; not: B = 6 (48 / 96) 26.7 / 23.3, 33.4 / 31.1, 39.3 / 35.0,
//     58.8 / 64.5; B = 12 (96 / 192) 31.1 / 28.6, 37.5 / 35.7, 47.9 / 53.7, 87.6 / 116; B = 20 (160 / 320) 31.9 / 29.7, 36.8 / 34.3, 55.9 / 64.6
//   ten, 70B, k = 18: B = 6 (144 / 240) 38.1 / 33.0, 49.4 / 35.0, 59.3 / 44.3, 106 / 97
//   twelve, 70B, k = 23: B = 1 (24 / 32) 31.2 / 28.7, 34.2 / 33.7, 37.2 / 34.9, 44.7 / 40.3; B = 8 (192 / 256) 43.6 / 35.6, 54.5 / 38.8, 72.2 / 53.7,
//     140 / 122; B = 14 (336 / 448) 48.2 / 44.7, 54.5 / 50.4, 91.0 / 82.3; not: B = 10 (240 / 320) 39.7 / 40.2, 43.7 / 44.7, 64.7 / 73.2, 155 / 176;
//     B = 20 (480 / 640) 57.2 / 60.3, 65.4 / 69.7, 109 / 115
//   fourteen, 70B, k = 27: B = 6 (192 / 240) 41.3 / 34.7, 52.4 / 37.9, 69.2 / 51.5, 137 / 115
static int attention_passes(int tiles, long heads)
{
    const int fewest = (tiles + MAX_TILES - 1) / MAX_TILES;
    if (tiles != 4 && (tiles < 10 || tiles > 15)) return fewest;
    auto one_round = [heads](int passes) { return heads * passes <= 256 && 256 / (heads * passes) * (heads * passes) > 192; };
    if (one_round(fewest + 1) || (heads * fewest > 256 && heads * (fewest + 1) <= 512)) return fewest + 1;
    return tiles == 10 && one_round(fewest + 2) ? fewest + 2 : fewest;
}

// Segments per sequence.  One workgroup per compute unit: what bounds a launch is the bytes that the busiest compute unit
// pulls, and every segment is a partial result of g*(k+1) rows to write and merge.  Two workgroups fit a compute unit; they are
// asked for where 256 leave a quarter of the device idle and the cache is passed over more than once.  sssd_op_attention over cold
// caches, us, all sequences at 3000 / at 1000..3000, by workgroups:
//   one pass, 8B: k = 8, B = 5: 240 35 / 33, 360 38 / 37, 480 38 / 37; B = 12: 192 50 / 47, 384 54 / 47, 480 53 / 48; B = 24: 192 68 / 62, 384 81 / 66;
//     k = 4, B = 20: 160 57 / 52, 320 72 / 59, 480 66 / 56; 70B, k = 0, B = 20: 160 59 / 55, 480 64 / 53
//   two passes: 70B, k = 8, B = 4: 256 42 / 41, 512 44 / 41; B = 9: 144 66 / 65, 432 61 / 55; B = 12: 192 67 / 66, 384 72 / 64; 8B, B = 10, k = 31:
//     160 79 / 78, 480 71 / 63; B = 12, k = 24: 192 79 / 78, 384 79 / 68; B = 16, k = 31, context 1000: 256 55, 512 67
// At least four blocks per segment, one for each wave; up to eight blocks are one segment, which is finished by its workgroup: its partial
// results and the merge's work cost more than the idle compute units, also where a cache with room has the merge launched.  One segment /
// segments of four blocks, caches of 4096, contexts 130 / 230: 8B B = 1, k = 0 17.0 / 18.9, 17.1 / 18.8, k = 8 22.2 / 22.5, 22.2 / 22.9; B = 4, k = 8
// 24.2 / 25.3, 24.5 / 25.9; B = 16, k = 4 24.6 / 27.1, 24.5 / 27.6; 70B B = 1, k = 8 29.0 / 29.3, 29.1 / 29.6; B = 4, k = 8 31.6 / 33.0, 31.8 / 33.6
// (without a merge launch, tiny shape, one sequence of 133 positions: step 73.5 -> 68.6 us).
AttnPlan attention_plan(const Dims &D, int B, int k)
{
    const int tiles = (D.g * (k + 1) + 15) / 16;
    AttnPlan p;
    p.passes = attention_passes(tiles, (long)B * D.nkv);
    const long units = (long)B * D.nkv * p.passes;   // workgroups for one segment of every sequence
    long share = 256 / units;
    if (p.passes > 1 && share * units <= 192) share = 512 / units;
    p.share = share < 1 ? 1 : (share > ATTN_MAX_SEGMENTS ? ATTN_MAX_SEGMENTS : (int)share);
    return p;
}

// The segments of a (sequence, kv head) are merged inside the launch where the groups are the same number on every die and no
// compute unit gets a second workgroup while others wait (two fit where the plan asks for two).
static bool attention_in_die(const Dims &D, const AttnPlan &p, int B)
{
    const long groups = (long)B * D.nkv * p.passes;
    const size_t slot_bytes = (size_t)round_up(D.g * (D.max_k + 1), 16) * D.d * sizeof(float);
    if (slot_bytes * p.share >= (size_t)1 << 31) return false;   // DieBuffer's offsets
    return B * D.nkv % 8 == 0 && groups <= HAND_GROUPS && groups * p.share <= 512;
}

static bool attention_merges(const Dims &D, const AttnPlan &p) { return p.share > 1 && D.blocks_per_seq > ATTN_WHOLE_BLOCKS; }

bool attention_hands_over(const Dims &D, const AttnPlan &p, int B) { return attention_merges(D, p) && attention_in_die(D, p, B); }

// Most partial results that any step of up to B sequences leaves, all kv heads.
size_t attention_slots(const Dims &D, int B)
{
    size_t most = 0;
    for (int b = 1; b <= B; ++b)
        for (int k = 0; k <= D.max_k; ++k) {
            const size_t n = (size_t)D.nkv * b * attention_plan(D, b, k).share;
            if (n > most) most = n;
        }
    return most;
}

hipError_t launch_attention(const Dims &D, const AttnArgs &a_in, hipStream_t s)
{
    AttnArgs a = a_in;
    const int q_rows_pad = round_up(D.g * (D.max_k + 1), 16);
    a.row_tiles = (D.g * (a.k + 1) + 15) / 16;
    a.plan = attention_plan(D, a.B, a.k);
    a.by_passes = Div(a.plan.passes);
    a.by_share = Div(a.plan.share);
    a.by_nkv = Div(D.nkv);
    a.by_g = Div(D.g);
    const bool merge = attention_merges(D, a.plan);
    if (!attention_hands_over(D, a.plan, a.B)) a.hand.words = nullptr;
    hipError_t e = D.d == 128 ? launch_partial<128>(D, a, q_rows_pad, s) : launch_partial<64>(D, a, q_rows_pad, s);
    if (e != hipSuccess) return e;
    // No merge where no sequence can have two segments.  With every workgroup of the merge returning at once the launch still
    // took 5 us (70B layer, B = 16, k = 8: 5 of 597; two layers of the tiny shape with room for 133 positions: 10 of 68).
    if (!merge || a.hand.words) return hipSuccess;
    const int n_tasks = a.B * D.nkv * D.g * (a.k + 1);
    if (D.d == 128) hipLaunchKernelGGL(attn_combine_kernel<128>, dim3((n_tasks + 3) / 4), dim3(256), 0, s, D, a, q_rows_pad);
    else hipLaunchKernelGGL(attn_combine_kernel<64>, dim3((n_tasks + 3) / 4), dim3(256), 0, s, D, a, q_rows_pad);
    return hipGetLastError();
}
