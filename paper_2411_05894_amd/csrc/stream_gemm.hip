// Weight-streaming GEMMs of the verify step and their fused epilogues.
//
// The linear rows of the paper's Table 2 (App. B) -- Q/K_new/V_new = X W, Y = A_out W_o,
// H = SwiGLU(Y W_1), Z = H W_2 -- and the LM head have FLOPs:IO ~ b*s_q, far below the
// MI355X ridge (~312 flop/byte), so each launch is a stream of the weight matrix through
// the matrix cores with everything else hidden behind it.
//
//   pgemm_kernel   M <= 32 rows (one or two 16-row tiles), as is_small has it.  Persistent: one workgroup of 16 waves per compute unit walks a
//                  list of 16-column output tiles.  Each wave owns a fixed k-slice and keeps the
//                  activations of that slice (bf16 hi and lo parts) in registers for the whole
//                  launch, so the inner loop touches memory only for weights.  Weight registers
//                  are refilled for the NEXT tile right after the MFMA that consumed them: a
//                  rolling prefetch with a constant number of bytes in flight per wave and no
//                  bubble at tile boundaries.  The k-split is reduced through LDS in fixed order.
//   qgemm16_kernel More rows (up to 160 at once, beyond in row blocks of 96 and 128 within one launch), and the matrices
//                  that is_small leaves to it.  v_mfma_f32_16x16x32_bf16 tiles: each wave of a workgroup of eight (four for the small
//                  matrices) owns 32 output columns and streams their weights HBM -> registers (rolling prefetch,
//                  every weight byte read once), while the activation k-tiles of the workgroup's k-slice, which all
//                  its waves need, are staged through a register ring and an LDS ring.  With the whole K in one
//                  workgroup it applies the epilogue itself; the slices of a split K are summed inside the launch, by
//                  workgroups of one die through its L2, or go to split-K partials for epi_kernel.
//   epi_kernel     Sums split-K partial results in fixed order and applies the epilogue, where they are not summed
//                  inside the launch: callers without a context, more workgroups than compute units.
//
// Epilogues (everything Table 2 leaves out is folded into them):
//   QKV     RMSNorm scale, rotary embedding, Q -> packed hi/lo operand, K/V -> cache (in place)
//   RESID   X += acc; packed X*gamma_next hi/lo; sums of squares per 16 or 32 columns, or per workgroup (nss_out says how many)
//   SWIGLU  RMSNorm scale, silu(gate)*up -> packed hi/lo operand
//   LM      RMSNorm scale, arg-max of a workgroup's columns (with an unsplit K logits are materialised only if asked for; else
//           they pass through memory once as unscaled sums)
// RMSNorm needs no pass of its own: the producer of the residual stream x writes x*gamma and
// partial sums of squares, the consuming GEMM scales its fp32 results by rsqrt(mean(x^2)+eps),
// which commutes with the matrix product.
#include "kernels.h"

#include <hip/hip_ext.h>

#include <type_traits>

#include "gemm_device.h"

namespace {

// ------------------------------------------------------------------ M <= 32 ----
constexpr int PW = 16;  // waves per workgroup

// Sums of squares of a row that an unsplit pgemm_kernel of KPW k-tiles per wave has room for, a whole number per lane: at most two for
// each of its PW * KPW k-tiles (seven per wave: 224, so four per lane and not three).
constexpr __host__ __device__ int small_row_sums(int kpw) { return (PW * kpw * 2 + 63) / 64 * 64; }

// A row of operand tiles as a buffer: the tile's place in it is a scalar, the lane's record the only vector part of the address.  With
// 64-bit vector addresses the first loads of a wave held forty registers.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_row(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00027000);
}
// Weight tile load.  One reader per byte (RH == 1): streaming, the line is not worth keeping.  Two
// workgroups of a die reading the same tiles (RH == 2): an ordinary load, so that the line is still in
// the die's L2 when the second request comes.
template <int AUX> __device__ __forceinline__ u32x4 load_tile(__amdgpu_buffer_rsrc_t row, int at, int lane)
{
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(row, lane * 16, at, AUX));
}
template <int RH> __device__ __forceinline__ u32x4 wload(__amdgpu_buffer_rsrc_t row, int at, int lane) { return load_tile<RH == 1 ? 2 : 0>(row, at, lane); }

template <int KPW, bool PREFETCH, int RH>
__device__ __forceinline__ f32x4 stream_tile(const u32x4 (&ah)[KPW], const u32x4 (&al)[KPW], u32x4 (&w)[KPW], __amdgpu_buffer_rsrc_t wn,
                                             const int (&koff)[KPW], int lane)
{
    f32x4 s0 = f32x4{0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
        s0 = mfma(ah[i], w[i], s0);
        s1 = mfma(al[i], w[i], s1);
        if (PREFETCH) {
            w[i] = wload<RH>(wn, koff[i], lane);
            __builtin_amdgcn_sched_barrier(0);   // here, not behind the last product: the compiler gathers them there, with one load left in flight
        }
    }
    return s0 + s1;
}

// grid = RH * n_groups * J workgroups of 1024 threads, each on one row tile of 16.  Workgroup
// (grp, j) computes its units over k-tiles [j*16*KPW, (j+1)*16*KPW); with J > 1 (SPLIT) it stores
// fp32 partial tiles, and the workgroup of a column group that arrives last sums them and applies the
// epilogue (epi_kernel does, in a second launch, when the launcher has no arrival counters for it).
// The unsplit instantiation carries none of that code (the QKV kernel is at the register limit).
//
// RH == 2 serves 17..32 rows without giving up the register-resident activations: the launch holds
// every workgroup twice, once for rows 0..15 and once for rows 16..31 (row tile rt), and the two copies
// sit 8 apart in the grid, i.e. on the same die, where they start together and ask for the same weight
// tiles: one of the two requests is served by the die's L2 (or merged with the other in flight), so
// HBM still sees each weight byte once (measured: 1.02 x the matrix bytes fetched per launch).
template <int EPI, int KPW, bool SPLIT, int RH, bool ONE>
__global__ __launch_bounds__(PW * 64) void pgemm_kernel(FusedGemmArgs a)
{
    constexpr int TPU = Unit<EPI>::TILES;
    __shared__ float red[2][PW][256];
    __shared__ float rstd_s[16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    // logical workgroup `bid` of `nblk`, and the row tile it serves
    int bid = blockIdx.x, nblk = gridDim.x, rt = 0;
    if (RH == 2) {
        nblk >>= 1;
        const int paired = nblk & ~7, b = blockIdx.x;           // whole sets of 8 logical workgroups, then the rest
        if (b < 2 * paired) {
            rt = (b >> 3) & 1;
            bid = ((b >> 4) << 3) | (b & 7);
        } else {
            const int rem = nblk - paired;
            rt = (b - 2 * paired) / rem;
            bid = paired + (b - 2 * paired) % rem;
        }
    }
    const int m_base = 16 * rt;
    const int J = SPLIT ? a.J : 1, j = SPLIT ? bid % J : 0, grp = SPLIT ? bid / J : bid;
    const int KT = a.KT;
    const int kt0 = (j * PW + wave) * KPW;
    // Units grp, grp + groups, grp + 2*groups, ... so that at any time the workgroups of a launch
    // read neighbouring tiles (measured 3 % faster on the layer matrices); the LM head, 30 times as
    // many tiles, measured 3 % faster with a contiguous run of upw units per workgroup.
    const int groups = nblk / J;
    constexpr bool RUNS = EPI == FEPI_LM;
    const int u_begin = RUNS ? grp * a.upw : grp, u_stride = RUNS ? 1 : groups;
    if (u_begin >= a.n_units) return;
    const int n_mine = RUNS ? (u_begin + a.upw < a.n_units ? a.upw : a.n_units - u_begin) : (a.n_units - grp + groups - 1) / groups;
    const int n_steps = n_mine * TPU;

    // k-tiles past the matrix (ragged K split) contribute zero activations and re-read the last tile; a wave that has no others reads
    // through buffers without records, which return zeros at once: of a K of 1040, 33 k-tiles, seven of sixteen waves (LM head of 128256
    // at two rows 47.6 -> 41.8 us).
    const int row_bytes = kt0 < KT ? KT * 1024 : 0;
    int koff[KPW];
#pragma unroll
    for (int i = 0; i < KPW; ++i) koff[i] = (kt0 + i < KT ? kt0 + i : KT - 1) * 1024;

    constexpr bool SCALED = EPI != FEPI_RESID && EPI != FEPI_STORE;
    u32x4 w[KPW], ah[KPW], al[KPW];
    const auto wp = tile_row(tile_weights<EPI>(a, unit_tile<EPI>(a, u_begin, 0)), row_bytes);
    const auto hi = tile_row(a.A_hi + (size_t)rt * KT * 64, row_bytes), lo = tile_row(a.A_lo + (size_t)rt * KT * 64, row_bytes);
    // Weights and activations of a k-tile together, in the order of their use: its products, and with them the request for the next
    // tile's weights, need not wait for the others.  No activation load under a branch: every wait would cover all of them.
    // A workgroup of one tile requests all its weights first: it has no next tile to request behind its products, and the last weights to
    // arrive bound it (8B O at nine rows 11.0 -> 10.0 us, LM head of 1024 9.2 -> 8.0).
    if (ONE) {
#pragma unroll
        for (int i = 0; i < KPW; ++i) {
            w[i] = wload<RH>(wp, koff[i], lane);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int i = 0; i < KPW; ++i) {
        if (!ONE) w[i] = wload<RH>(wp, koff[i], lane);
        ah[i] = load_tile<0>(hi, koff[i], lane);
        al[i] = load_tile<0>(lo, koff[i], lane);
        __builtin_amdgcn_sched_barrier(0);
    }
    // What bounds it: the weight stream, 8 TB/s once it runs (8B gate/up, 235 MB), and in front of it the chain from the launch to the
    // first products, 7-10 us of a 9-25 us launch.  The operands of a k-tile are therefore requested together and in the order of use, none
    // under a branch, and nothing else in front of them: 8B step of nine rows 3295 -> 3261 us.
    // The row scales are needed by the first epilogue only: their sums (wave w: of row w) are requested behind the operands and added up
    // behind the first tile's products, so no load of the first tiles waits for them.  (QKV at eight k-tiles per wave, four sums per lane: seven
    // registers spilled at the limit of 128, ten accesses in a workgroup's life; 13.6 us, 14.4 with the sums added up in front and four spilled.)
    constexpr int SV = small_row_sums(KPW) / 64;   // per lane
    float sv[SV];
    const int ms = m_base + wave < a.M ? m_base + wave : a.M - 1;
    if (SCALED && !SPLIT) {
        const float *p = a.ssq_in + (size_t)ms * a.nss_in;
#pragma unroll
        for (int i = 0; i < SV; ++i) sv[i] = p[lane + 64 * i < a.nss_in ? lane + 64 * i : 0];
        __builtin_amdgcn_sched_barrier(0);
    }

    // ... and what the only epilogue of a workgroup adds to
    constexpr bool AHEAD = ONE && EPI == FEPI_RESID && !SPLIT;
    float x_ahead = 0.f;
    uint16_t g_ahead = 0;
    if (AHEAD) {
        const int m = m_base + 4 * (lane >> 4) + (wave & 3), n = u_begin * 16 + (lane & 15);
        x_ahead = a.X[(size_t)(m < a.M ? m : a.M - 1) * a.h + n];
        g_ahead = a.gamma_next[n];
        __builtin_amdgcn_sched_barrier(0);
    }

    if (kt0 + KPW > KT) {
#pragma unroll
        for (int i = 0; i < KPW; ++i)
            if (kt0 + i >= KT) ah[i] = al[i] = u32x4{0, 0, 0, 0};
    }

    float keep = 0.f;
    Best best = Best::none();   // LM: of this thread's row and column within the tiles
    auto scales = [&]() {
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < SV; ++i) sum += lane + 64 * i < a.nss_in ? sv[i] : 0.f;
        sum = wave_sum(sum);
        if (lane == 0) rstd_s[wave] = rsqrtf(sum / (float)a.h + a.eps);
    };
    auto step = [&](int s, auto first, auto more) {
        constexpr bool SCALES = decltype(first)::value && SCALED && !SPLIT, MORE = decltype(more)::value;
        const int unit = u_begin + (s / TPU) * u_stride, part = s % TPU;
        const int next = MORE && s + 1 < n_steps ? s + 1 : s;
        const auto wn = tile_row(tile_weights<EPI>(a, unit_tile<EPI>(a, u_begin + (next / TPU) * u_stride, next % TPU)), row_bytes);
        const f32x4 acc = stream_tile<KPW, MORE, RH>(ah, al, w, wn, koff, lane);
        if (SCALES) scales();
        float *rb = &red[s & 1][0][0];
#pragma unroll
        for (int r = 0; r < 4; ++r) rb[wave * 256 + r * 64 + lane] = acc[r];
        __syncthreads();
        // Buffer s&1 is rewritten at step s+2, after the barrier of step s+1, which the reducing waves
        // reach only after they have read it.
        if (wave < 4) {
            float v = 0.f;
#pragma unroll
            for (int ww = 0; ww < PW; ++ww) v += rb[ww * 256 + wave * 64 + lane];
            const int ml = 4 * (lane >> 4) + wave, m = m_base + ml, c = lane & 15;
            if (SPLIT) {
                // device-scope: read back by the last workgroup of the group, on whichever die it runs
                st<true>(a.partials + ((size_t)j * a.part_rows + m) * a.Ntot + unit_tile<EPI>(a, unit, part) * 16 + c, v);
            } else if (TPU == 2 && part == 0) {
                keep = v;
            } else {
                const float rs = (EPI == FEPI_RESID || EPI == FEPI_STORE) ? 1.f : rstd_s[ml];
                if (EPI == FEPI_LM) {
                    const int n = unit * 16 + c;
                    best.take(v * rs, n);
                    if (m < a.M && a.logits) a.logits[(size_t)m * a.vocab + n] = v * rs;
                } else if (AHEAD) resid1<false>(a, unit, m, c, m < a.M, v, x_ahead, g_ahead);
                else if (TPU == 2) epilogue<EPI>(a, unit, m, c, m < a.M, keep, v, rs);
                else epilogue<EPI>(a, unit, m, c, m < a.M, v, 0.f, rs);
            }
        }
    };
    // Steps with and without a next tile apart: where both meet, a wait covers the next tile's loads.  A workgroup with fewer tiles than
    // the others (ONE: all have one) may fetch its only one twice.
    step(0, std::true_type{}, std::integral_constant<bool, !ONE>{});
    if (!ONE) {
        for (int s = 1; s + 1 < n_steps; ++s) step(s, std::false_type{}, std::true_type{});
        if (n_steps > 1) step(n_steps - 1, std::false_type{}, std::false_type{});
    }

    if (EPI == FEPI_LM && !SPLIT && wave < 4) {
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) best.across(off);
        const int m = m_base + 4 * (lane >> 4) + wave;
        if (m < a.M && (lane & 15) == 0) {
            a.part_val[(size_t)m * a.n_part + grp] = best.v;
            a.part_idx[(size_t)m * a.n_part + grp] = best.i;
        }
    }

    // Split K with arrival counters: the workgroup of a (row tile, column group) that finishes last
    // sums the group's slices (in slice order, so the result does not depend on which one that is)
    // and applies the epilogue -- no second launch.  The slices were stored device-scope and each wave
    // waits for its stores before the workgroup is counted; they are read back device-scope.  The
    // counter is back at zero for the next launch on the stream.
    if (SPLIT && a.tail_count) {
        __shared__ int last_s;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) {
            int *count = a.tail_count + rt * groups + grp;
            const int old = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last_s = old == J - 1;
            if (old == J - 1) __hip_atomic_store(count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!last_s) return;
        if (SCALED) {
            rstd_s[wave] = row_rstd(a, m_base + wave, lane);
            __syncthreads();
        }
        if (EPI == FEPI_RESID) {
            // thread for thread what epi_kernel does (same order of every sum): a wave takes two units,
            // 8 columns per thread, lanes 16 apart share a unit's sum of squares
            const int r = lane & 15, kg = lane >> 4;
            for (int i = 2 * wave + (kg >> 1); i - (kg >> 1) < n_mine; i += 2 * PW) {
                const int unit = u_begin + i * u_stride, col = unit * 16 + (kg & 1) * 8;
                const int m = m_base + r;
                const bool live = i < n_mine && m < a.M;
                Vec8 v0{};
                if (live) sum_slices<4, false, true>(a, m, col, 0, v0, v0);
                resid_block<false>(a, m, col, live, kg, v0);
            }
        } else {
            const size_t jstride = (size_t)a.part_rows * a.Ntot;
            for (int e = threadIdx.x; e < n_mine * 256; e += PW * 64) {   // 16 adjacent lanes: one row of a unit
                const int unit = u_begin + (e >> 8) * u_stride, ml = (e & 255) >> 4, m = m_base + ml, c = e & 15;
                float v[TPU];
#pragma unroll
                for (int part = 0; part < TPU; ++part) {
                    const float *pp = a.partials + (size_t)m * a.Ntot + unit_tile<EPI>(a, unit, part) * 16 + c;
                    float sum = ld<true>(pp);
                    for (int jj = 1; jj < J; ++jj) sum += ld<true>(pp + jj * jstride);
                    v[part] = sum;
                }
                if (EPI == FEPI_LM) {
                    const float logit = v[0] * rstd_s[ml];
                    best.take(logit, unit * 16 + c);
                    if (m < a.M && a.logits) a.logits[(size_t)m * a.vocab + unit * 16 + c] = logit;
                } else {
                    epilogue<EPI>(a, unit, m, c, m < a.M, v[0], TPU == 2 ? v[TPU - 1] : 0.f, SCALED ? rstd_s[ml] : 1.f);
                }
            }
            if (EPI == FEPI_LM) {   // every fourth tile of a row lies with the threads 256 on
                __shared__ Best best_s[4][16];
#pragma unroll
                for (int off = 8; off >= 1; off >>= 1) best.across(off);
                if ((threadIdx.x & 15) == 0) best_s[threadIdx.x >> 8][(threadIdx.x & 255) >> 4] = best;
                __syncthreads();
                const int m = m_base + threadIdx.x;
                if (threadIdx.x < 16 && m < a.M) {
                    Best all = best_s[0][threadIdx.x];
#pragma unroll
                    for (int x = 1; x < 4; ++x) all.take(best_s[x][threadIdx.x].v, best_s[x][threadIdx.x].i);
                    a.part_val[(size_t)m * a.n_part + grp] = all.v;
                    a.part_idx[(size_t)m * a.n_part + grp] = all.i;
                }
            }
        }
    }
}

// ---- epilogue from split-K partials ----
// The same four epilogues on 8 consecutive output columns per thread: thread (row r = lane%16,
// column group kg = lane/16) of a wave owns columns 8*kg..8*kg+7 of a 32-column block, which is
// exactly one 16-byte lane record of the packed operand layout, so a wave writes whole operand
// tiles (1 KiB, contiguous) and reads 128 contiguous bytes of each partial row.
// Column blocks of 32 per epilogue: plain output columns, except QKV, whose blocks run over the
// first-half channels of each head (the rotary partner columns come along).
template <int EPI> __device__ __host__ __forceinline__ int column_blocks(const FusedGemmArgs &a)
{
    if (EPI == FEPI_QKV) return (a.nq + 2 * a.nkv) * ((a.d / 2 + 31) / 32);
    if (EPI == FEPI_SWIGLU) return (a.Ntot / 2 + 31) / 32;
    return (a.Ntot + 31) / 32;
}

// grid = (column-block groups, row tiles of 16), 256 threads; each wave takes column blocks
// cb0 + wave, cb0 + wave + 4, ...  The partial sums of the first block are fetched before the row scales are reduced, two slices at
// a time: the waves of a compute unit hide the round trips better than a wave's own loads do.  Eight slices at a time (four, of two
// columns) took 118-127 registers and four workgroups per compute unit, two take 42-85 and five to eight fit: RESID of 160 rows x 4096 in
// four slices 11.8 -> 10.4 us, in seven 8.0 -> 7.3, of 144 rows x 8192 11.5 -> 10.5, QKV of 160 rows 11.3 -> 10.4, of 36 rows 8.1 -> 7.7, of 512
// rows 15.7 -> 14.6; one at a time the same or up to 5 % slower.  A second block of a wave, in wide outputs at many rows, is
// not fetched ahead: with eight slices that had taken 129-143 registers and a second, quarter-full round of workgroups at 512 rows (RESID
// 12.8 -> 11.9 us without).  RESID leaves one sum of squares per row and workgroup: the launches that scale rows read few of them.
template <int EPI>
__global__ __launch_bounds__(256) void epi_kernel(FusedGemmArgs a, int blocks_per_wg)
{
    __shared__ float rstd_s[16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m0 = blockIdx.y * 16;
    constexpr bool SCALED = EPI != FEPI_RESID && EPI != FEPI_STORE;
    constexpr bool PAIRED = EPI == FEPI_QKV || EPI == FEPI_SWIGLU;
    const int r = lane & 15, kg = lane >> 4, m = m0 + r;
    const bool row_ok = m < a.M;
    const int n_cb = column_blocks<EPI>(a);
    const int cb_begin = blockIdx.x * blocks_per_wg;
    const int cb_end = cb_begin + blocks_per_wg < n_cb ? cb_begin + blocks_per_wg : n_cb;
    const int half = a.d >> 1, bph = (half + 31) / 32;   // QKV: column blocks per head

    // first output column of this thread in block cb (QKV: of the head's first half), or -1
    auto column = [&](int cb) -> int {
        if (!row_ok) return -1;
        if (EPI == FEPI_QKV) {
            const int ch = (cb % bph) * 32 + kg * 8;
            return ch < half ? (cb / bph) * a.d + ch : -1;
        }
        const int n0 = cb * 32 + kg * 8;
        return n0 < (EPI == FEPI_SWIGLU ? a.Ntot >> 1 : a.Ntot) ? n0 : -1;
    };
    auto fetch = [&](int cb, Vec8 &v0, Vec8 &v1) {
        const int col = cb < cb_end ? column(cb) : -1;
        if (col >= 0) {
            sum_slices<2, PAIRED>(a, m, col, col + (EPI == FEPI_QKV ? half : a.Ntot >> 1), v0, v1);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v0.v[e] = v1.v[e] = 0.f;
        }
    };

    // Row scales: four rows per wave.  Their loads go out first and the first block's partial
    // sums right behind them, so the two dependent round trips overlap.
    constexpr int SV = 2;                     // sums of squares per lane and row held in registers: all that a launch of this kernel leaves
    const int NSS = a.nss_in;
    float sv[4][SV];
    if (SCALED) {   // no load under a branch: each would be waited for by itself
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int mm = m0 + wave + 4 * q;
            const float *p = a.ssq_in + (size_t)(mm < a.M ? mm : a.M - 1) * NSS;
#pragma unroll
            for (int i = 0; i < SV; ++i) sv[q][i] = p[lane + 64 * i < NSS ? lane + 64 * i : 0];
        }
    }
    Vec8 v0, v1;
    fetch(cb_begin + wave, v0, v1);
    if (SCALED) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int mm = m0 + wave + 4 * q;
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < SV; ++i) sum += lane + 64 * i < NSS ? sv[q][i] : 0.f;
            if (mm < a.M)
                for (int t = lane + 64 * SV; t < NSS; t += 64) sum += a.ssq_in[(size_t)mm * NSS + t];
            sum = wave_sum(sum);
            if (lane == 0) rstd_s[wave + 4 * q] = rsqrtf(sum / (float)a.h + a.eps);
        }
        __syncthreads();
    }
    const float rs = SCALED ? rstd_s[r] : 1.f;

    float ss = 0.f;   // RESID: of this row, over the thread's columns
    Best best = Best::none();   // LM: likewise
    for (int cb = cb_begin + wave; cb < cb_end; cb += 4) {
        if (cb != cb_begin + wave) fetch(cb, v0, v1);
        const int col = column(cb);
        const bool live = col >= 0;
        if (EPI == FEPI_QKV) {
            if (live) qkv8(a, m, cb / bph, col - (cb / bph) * a.d, rs, v0, v1);   // first-half channel of v0[0]
        } else if (EPI == FEPI_SWIGLU) {
            if (live) swiglu8(a, m, col, rs, v0, v1);
        } else if (EPI == FEPI_STORE) {
            if (live) store8(a.out + (size_t)m * a.Ntot + col, v0);
        } else if (EPI == FEPI_RESID) {
            if (live) ss += resid8<false>(a, m, col, v0);
        } else {  // FEPI_LM
            if (live) lm8(a, m, col, rs, v0, best);
        }
    }
    if (EPI == FEPI_LM) {   // one arg-max per row and workgroup
        __shared__ Best best_s[4][16];
        best.across(16);
        best.across(32);
        if (kg == 0) best_s[wave][r] = best;
        __syncthreads();
        if (threadIdx.x < 16 && row_ok) {
#pragma unroll
            for (int x = 1; x < 4; ++x) best.take(best_s[x][r].v, best_s[x][r].i);
            a.part_val[(size_t)m * gridDim.x + blockIdx.x] = best.v;
            a.part_idx[(size_t)m * gridDim.x + blockIdx.x] = best.i;
        }
    }
    if (EPI == FEPI_RESID) {   // one sum of squares per row and workgroup
        __shared__ float ss_s[4][16];
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        if (kg == 0) ss_s[wave][r] = ss;
        __syncthreads();
        if (threadIdx.x < 16 && row_ok)
            a.ssq_out[(size_t)m * gridDim.x + blockIdx.x] = (ss_s[0][r] + ss_s[1][r]) + (ss_s[2][r] + ss_s[3][r]);
    }
}

template <int EPI> hipError_t launch_epi(FusedGemmArgs &a, hipStream_t s)
{
    const int n_cu = a.n_cu > 0 ? a.n_cu : 256;
    const int row_tiles = (a.M + 15) / 16;
    const int n_cb = column_blocks<EPI>(a);
    // about 4 workgroups per compute unit, whole groups of four column blocks (one per wave)
    const int groups_x = (4 * n_cu + row_tiles - 1) / row_tiles;
    int bpw = (n_cb + groups_x - 1) / groups_x;
    bpw = (bpw + 3) / 4 * 4;
    const int nx = (n_cb + bpw - 1) / bpw;
    if (EPI == FEPI_RESID) a.nss_out = nx;
    if (EPI == FEPI_LM) a.n_part = nx;
    hipLaunchKernelGGL((epi_kernel<EPI>), dim3(nx, row_tiles), dim3(256), 0, s, a, bpw);
    return hipGetLastError();
}

// ------------------------------------------------------------------- M > 32 ----
// Packed weights of concatenated 16-column tile gt for any epilogue: the output is up to three
// matrices side by side, the first two of seg0 and seg1 tiles.
__device__ __forceinline__ const u32x4 *tile_weights_seg(const FusedGemmArgs &a, int gt)
{
    const size_t stride = (size_t)a.KT * 64;
    const u32x4 *base = a.W0;
    if (gt >= a.seg0) {
        gt -= a.seg0;
        base = a.W1;
        if (gt >= a.seg1) {
            gt -= a.seg1;
            base = a.W2;
        }
    }
    return base + gt * stride;
}

// Concatenated 16-column tile at place t of the order in which the waves take them.  WHOLE: the two tiles of an epilogue unit (rotary
// partners, gate and up) side by side, so that one wave holds both.  Else any order serves; gate and up side by side measured
// 14.5 against 16.7-17.4 us for 2 x 8192 columns of K = 2048 at 20 rows (8B gate/up at 65..80 rows 50 against 47, at 160 rows the same).
template <bool WHOLE> __device__ __forceinline__ int q_tile(const FusedGemmArgs &a, int t)
{
    if (a.epi == FEPI_SWIGLU) return unit_tile<FEPI_SWIGLU>(a, t >> 1, t & 1);
    if (WHOLE && a.epi == FEPI_QKV) return unit_tile<FEPI_QKV>(a, t >> 1, t & 1);
    return t;
}

// rsqrt(mean(x^2) + eps) of ROWS rows from m0 on into LDS (published by the caller's barrier), 16 lanes a row: request() goes in
// front of the launch's first operands, finish() behind them.
template <int ROWS, int QW> struct RowScales {
    static constexpr int TURNS = ROWS / (4 * QW) + (ROWS % (4 * QW) != 0);   // rows per lane
    static constexpr int U = TURNS > 4 ? 4 : 16 / TURNS;                     // sums per lane and row in flight
    float v[TURNS][U];
    __device__ __forceinline__ void load(const float *sums, int n, int M, int m0, int t0)
    {
#pragma unroll
        for (int i = 0; i < TURNS; ++i) {
            const int m = m0 + (threadIdx.x >> 4) + i * 4 * QW;
            const float *p = sums + (size_t)(m < M ? m : M - 1) * n;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + (threadIdx.x & 15) + 16 * u;
                v[i][u] = p[t < n ? t : 0];
            }
        }
    }
    __device__ __forceinline__ void add(int n, int t0, float (&sum)[TURNS])
    {
#pragma unroll
        for (int i = 0; i < TURNS; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) sum[i] += t0 + (int)(threadIdx.x & 15) + 16 * u < n ? v[i][u] : 0.f;
    }
    // Without `scaled` (no sums to read) it loads activations for nothing: under a branch the first sum, and so the wait for it, comes
    // before the first operands are requested (1 us of 1B..70B gate/up launches).
    __device__ __forceinline__ void request(const FusedGemmArgs &a, int m0, bool scaled)
    {
        load(scaled ? a.ssq_in : reinterpret_cast<const float *>(a.A_hi), scaled ? a.nss_in : 1, a.M, m0, 0);
    }
    template <typename Args> __device__ __forceinline__ void finish(const Args &a, int m0, float *rstd_s)
    {
        float sum[TURNS];
#pragma unroll
        for (int i = 0; i < TURNS; ++i) sum[i] = 0.f;
        add(a.nss_in, 0, sum);
        for (int t0 = 16 * U; t0 < a.nss_in; t0 += 16 * U) {
            load(a.ssq_in, a.nss_in, a.M, m0, t0);
            add(a.nss_in, t0, sum);
        }
#pragma unroll
        for (int i = 0; i < TURNS; ++i) {
            const int r = (threadIdx.x >> 4) + i * 4 * QW;
            const float total = row16_sum(sum[i]);
            if (r < ROWS && (threadIdx.x & 15) == 0) rstd_s[r] = rsqrtf(total / (float)a.h + a.eps);
        }
    }
};

// grid = row blocks * column groups * J workgroups of QW waves on MT16 row tiles of 16.
// Weights are the first operand of the products and activations the second, so a lane ends with four consecutive columns of one row: the
// epilogues work on the accumulators as they are, store quads, and two lanes swap halves where a whole operand record is wanted (stored by
// halves every line is written twice, 2 us of a launch).  Through LDS, with eight columns per lane, the epilogues cost 2-4 us more:
// 70B layer at 144 rows 570 -> 561 us a step, two 8B layers at 512 rows 950 -> 939, at 160 rows 544 -> 527.
// A whole K (J = 1) is finished by its workgroup.  As a launch of its own behind sums in memory the epilogue cost 70B gate/up at 144 rows
// 16.6 us, 8B gate/up at 512 rows 24 us, an LM head of 128256 at 91 rows 27 us.
// Both operands are the packed tiles as stored: lane l holds (row or column l%16, k-slots 8*(l/16)..+7) of a 16 x 32 tile.
// The three forms (QForm) have kernels of their own: the epilogue's row scales and tile order in front of the first loads, and its
// staging area, cost the split GEMMs that use none of it 0.3-1 us each -- 4096 x 4096 at 36 rows 13.3 -> 12.4 us, 8B QKV at 36 rows
// 14.6 -> 13.5, K = 1024 at 33 rows 7.7 -> 6.9; steps of 33..160 rows 0.5-4 %.
// The first loads go out in the order of the loop (sched_barrier): reordered by the compiler they make the wait at the top of some loops
// drain what is in flight once every QDW k-tiles (8B gate/up at 36 rows: loop 49.8 -> 42 us).  QDW = 4: with 3 / 6 / 8 weight k-tiles in
// flight two 8B layers at 36 rows and 32768 positions take 426 / 425 / 428 us instead of 422, at 25 rows 237 instead of 232 with 3.
// One 32-column tile pair per wave, so two waves share a SIMD at QW = 8 (256 columns per workgroup, the large matrices);
// QW = 4 for the small ones, whose K then splits half as often.
//
// What bounds it: below about 100 rows the weight stream, above that the matrix pipes, which at 512 rows are busy 70 % of
// the cycles of a compute unit that has work (and the clock falls to 2.0 GHz under that load); the rest goes into operand
// reads, stores and barriers between the MFMAs.  So the instruction stream of a k-tile is fixed by hand: operand
// tiles are read from LDS AHEAD MFMA groups before their use, straight across the k-tile boundary; the chunk of the next
// k-tile is stored early in the current one, and the barrier that publishes it stands just before the first read of it,
// so that waves may be most of a k-tile apart without waiting and no read latency follows a barrier.  Left to the
// compiler, most reads were issued right before their use.  Measured against that form, GEMM and epilogue, us: 8B gate/up
// 160 rows 84 -> 82, 512 rows 240 -> 234; 70B gate/up 144 rows 274 -> 262, 512 rows 894 -> 850; 70B down 144 rows 147 -> 135.
// Against v_mfma_f32_32x32x16_bf16, which 33..48 rows used to take: 8B 36 rows gate/up 48.7 -> 45.3, down 32.4 -> 29.4,
// 70B gate/up 157 -> 147.
//
// More than 160 rows are cut into blocks of eight or six row tiles, all in one launch: blocks 8 apart in the grid run on one
// die, where the row blocks of a (column group, slice) follow each other and share the weights through its L2 (ordinary
// loads then, not streaming ones).  There the matrix pipes bound everything and two waves share 64 columns, each on half
// of the rows: half the operand reads per MFMA for a second fetch of the weights from the die's L2 (8B gate/up at 512 rows
// 235 -> 220 us, but 84 -> 100 us at 160 rows, which are still bound by what a compute unit can fetch).
// What becomes of a workgroup's sums: they are stored for epi_kernel, they are whole and go through the epilogue here, or they are
// handed over to the workgroups of the same columns and rows, which share the units of the epilogue out.  The last form holds four
// epilogues, each for a share and for the whole of the work, unrolled: 8-21 thousand instructions, run through once, with 70-200 scalars kept in
// vector registers; 4-9 us lie between a workgroup's last product and its last store.
enum QForm { PARTS, WHOLE, DIE };
template <int MT16, int QW, bool BLOCKS, int FORM> struct QShape {
    static constexpr int QDW = BLOCKS ? 3 : 4;                  // k-tiles in flight
    static constexpr int TILES = MT16 * 2;                      // activation tiles (hi and lo) of one k-tile
    static constexpr int APT = (TILES + QW - 1) / QW;           // tiles fetched per wave; surplus waves re-read the last one
    static constexpr int SLOT = TILES * 64;                     // records of a ring slot
    static constexpr int RING = QDW * SLOT, STAGE = FORM == PARTS ? 0 : QW * 8 * (FORM == DIE ? MT16 : MT16 / (BLOCKS ? 2 : 1));   // records of the ring, of the waves' row sums or maxima
    static constexpr int LDS = RING > STAGE ? RING : STAGE;
};

// What qgemm16_kernel's epilogues read of FusedGemmArgs, its first argument: these fields and no others, so an epilogue that needs one more
// does not compile before it is named here.
#define SSSD_EPILOGUE_VALUES(V)                                                                                                        \
    V(M) V(h) V(d) V(nq) V(nkv) V(k) V(q_rows_pad) V(vocab) V(eps) V(nss_in) V(nss_out) V(KT_out) V(n_part) V(Ntot) V(J) V(epi)
#define SSSD_EPILOGUE_POINTERS(P)                                                                                                      \
    P(X) P(ssq_out) P(out_hi) P(out_lo) P(Qp) P(Qp_lo) P(Kc) P(Vc) P(logits) P(part_val) P(part_idx) P(out) P(ssq_in) P(gamma_next)    \
    P(rope_cs) P(pos_base) P(rope_pos)
struct EpilogueArgs {
#define SSSD_FIELD(f) decltype(FusedGemmArgs::f) f;
    SSSD_EPILOGUE_VALUES(SSSD_FIELD)
    SSSD_EPILOGUE_POINTERS(SSSD_FIELD)
#undef SSSD_FIELD
    Div by_J, by_k1, by_g;
    KvGeom kv;
    Hand hand;
};

// Loaded where it is called: loaded in front of the main loop, as the compiler does by itself, these sixty scalars are moved into
// vector registers and back (130 instructions in front of the first load).
__device__ __forceinline__ EpilogueArgs epilogue_arguments()
{
    using Constant = const __attribute__((address_space(4))) FusedGemmArgs;
    Constant *p = (Constant *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));   // not before
    EpilogueArgs e;
#define SSSD_VALUE(f) e.f = p->f;
#define SSSD_POINTER(f) e.f = (decltype(e.f))(__attribute__((address_space(1))) const void *)(const void *)p->f;
    SSSD_EPILOGUE_VALUES(SSSD_VALUE)
    SSSD_EPILOGUE_POINTERS(SSSD_POINTER)
    // member by member, all of them: there is no copy out of constant memory
    static_assert(sizeof(Div) == 8 && sizeof(KvGeom) == 24 && sizeof(Hand) == 24, "every member is loaded below");
    SSSD_VALUE(by_J.d) SSSD_VALUE(by_J.m) SSSD_VALUE(by_k1.d) SSSD_VALUE(by_k1.m) SSSD_VALUE(by_g.d) SSSD_VALUE(by_g.m)
    SSSD_POINTER(kv.table) SSSD_VALUE(kv.blocks_per_seq) SSSD_VALUE(kv.n_pages) SSSD_VALUE(kv.nkv) SSSD_VALUE(kv.d)
    SSSD_POINTER(hand.words) SSSD_POINTER(hand.parts) SSSD_VALUE(hand.polls)
#undef SSSD_VALUE
#undef SSSD_POINTER
    return e;
}
#undef SSSD_EPILOGUE_VALUES
#undef SSSD_EPILOGUE_POINTERS

// Rows 16 * tile0 .. 16 * (tile0 + MT16) - 1, column group grp, slice j; set: the group of workgroups that hand over to each other (DIE).
template <int MT16, int QW, bool BLOCKS, int FORM>
__device__ __forceinline__ void qgemm16_rows(const FusedGemmArgs a, int NT16, int tile0, int grp, int j, int set, u32x4 *lds, float *rstd_s)
{
    using S = QShape<MT16, QW, BLOCKS, FORM>;
    constexpr bool PAIRS = FORM != PARTS;    // a wave holds both tiles of an epilogue unit
    u32x4 (*ring)[S::SLOT] = reinterpret_cast<u32x4 (*)[S::SLOT]>(lds);
    constexpr int QDW = S::QDW, TILES = S::TILES, APT = S::APT;
    constexpr bool TWO = BLOCKS || MT16 <= 3;     // sums in two levels, where the registers allow it
    constexpr bool COMP = !BLOCKS && MT16 <= 2;   // ... the upper one compensated
    constexpr int RH = BLOCKS ? 2 : 1;       // waves that share a column group, each on its part of the rows
    static_assert(MT16 % RH == 0, "every wave has the same number of row tiles");
    constexpr int CW = QW / RH;                   // column groups per workgroup
    constexpr int NC = 2 * RH;                    // 16-column tiles per wave
    constexpr int MTW = MT16 / RH;                // row tiles per wave
    constexpr int RECS = 2 * MTW;                 // operand tiles every wave reads per k-tile
    constexpr int AHEAD = (RECS - 1) / 2 < 6 ? (RECS - 1) / 2 : 6;   // of them read before their use
    constexpr int BAR = RECS - AHEAD;             // the first read of the next k-tile
    constexpr int PUT = BAR - AHEAD - 1;          // chunk stores: at least AHEAD reads lie between them and the barrier
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int half = wave / CW, cg = wave % CW;
    const int m_base = tile0 * 16;
    const int KT = a.KT;
    const int kps = a.kps;
    const int kt_begin = j * kps, kt_end = kt_begin + kps < KT ? kt_begin + kps : KT;
    const int n_iter = kt_end - kt_begin;

    const int c16 = (grp * CW + cg) * NC;         // this wave's first 16-column tile, in the order of q_tile
    const u32x4 *wp[NC];
#pragma unroll
    for (int ct = 0; ct < NC; ++ct)               // columns past the matrix re-read the last tile, never stored
        wp[ct] = tile_weights_seg(a, q_tile<PAIRS>(a, c16 + ct < NT16 ? c16 + ct : NT16 - 1)) + lane;
    const u32x4 *asrc[APT];
#pragma unroll
    for (int i = 0; i < APT; ++i) {
        int t = wave + i * QW;                    // row tile t / 2, part t % 2 (0: hi, 1: lo)
        if (t >= TILES) t = TILES - 1;
        int rt = tile0 + (t >> 1);
        if (rt >= a.part_rows >> 4) rt = (a.part_rows >> 4) - 1;   // past the rows: never stored
        asrc[i] = ((t & 1) ? a.A_lo : a.A_hi) + (size_t)rt * KT * 64 + lane;
    }
    f32x4 acc[MTW][NC], total[MTW][NC], lost[MTW][NC];
#pragma unroll
    for (int i = 0; i < MTW; ++i)
#pragma unroll
        for (int ct = 0; ct < NC; ++ct) acc[i][ct] = total[i][ct] = lost[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};

    u32x4 w[QDW][NC], apre[QDW][APT];
    auto load_a = [&](int u, int it) {
        const size_t kt = (size_t)(kt_begin + (it < n_iter ? it : n_iter - 1)) * 64;
#pragma unroll
        for (int i = 0; i < APT; ++i) apre[u][i] = asrc[i][kt];
    };
    auto load_w = [&](int u, int it) {
        const size_t kt = (size_t)(kt_begin + (it < n_iter ? it : n_iter - 1)) * 64;
#pragma unroll
        for (int ct = 0; ct < NC; ++ct) w[u][ct] = BLOCKS ? wp[ct][kt] : __builtin_nontemporal_load(wp[ct] + kt);
    };
    auto stage = [&](int u) {
#pragma unroll
        for (int i = 0; i < APT; ++i)   // without the padding: at nine tiles and eight waves a quarter of the stores
            if (TILES % QW == 0 || i < APT - 1 || wave + i * QW < TILES) ring[u][(wave + i * QW) * 64 + lane] = apre[u][i];
    };
    const bool scaled = FORM != PARTS && a.epi != FEPI_RESID && a.epi != FEPI_STORE;
    RowScales<16 * MT16, QW> scales;
    if (FORM == WHOLE) scales.request(a, m_base, scaled);
#pragma unroll
    for (int u = 0; u < QDW; ++u) {
        load_a(u, u);
        load_w(u, u);
        __builtin_amdgcn_sched_barrier(0);   // in the order of the loop: what the first turn may leave in flight, every turn may
    }
    if (FORM == WHOLE && scaled) scales.finish(a, m_base, rstd_s);
    __builtin_amdgcn_sched_barrier(0);
    stage(0);
    __syncthreads();
    const int a_at = half * MTW * 128 + lane;
    u32x4 x[RECS + AHEAD];
#pragma unroll
    for (int r = 0; r < AHEAD; ++r) x[r] = ring[0][a_at + r * 64];

    auto ktile = [&](int u, int it, bool refill) {
        const int un = (u + 1) % QDW;
#pragma unroll
        for (int r = 0; r < RECS; ++r) {
            if (r == BAR) {
                // lgkmcnt counts LDS operations in order: with at least AHEAD reads issued since the stores of the next
                // chunk, AHEAD or fewer outstanding means that the stores are done.
                asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(AHEAD) : "memory");
                asm volatile("s_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
            x[r + AHEAD] = r < BAR ? ring[u][a_at + (r + AHEAD) * 64] : ring[un][a_at + (r + AHEAD - RECS) * 64];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ct = 0; ct < NC; ++ct) acc[r >> 1][ct] = mfma(w[u][ct], x[r], acc[r >> 1][ct]);
            __builtin_amdgcn_sched_barrier(0);
            if (r == PUT) {
                stage(un);
                if (refill) load_a(u, it + QDW);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (refill) load_w(u, it + QDW);
#pragma unroll
        for (int r = 0; r < AHEAD; ++r) x[r] = x[RECS + r];
    };
    // A running fp32 sum over hundreds of k-tiles loses more bits than sums of a few k-tiles and a sum of those, which the
    // register-resident kernel and the deeper K splits of four passes had for free.  Relative error against 64 bits, one
    // level / two: 70B down at 32 rows 7.7e-7 / 1.8e-7, at 512 rows 1.1e-6 / 2.0e-7 (passes 5.8e-7).  Up to 32 rows, which
    // share their sizes with pgemm_kernel, the sum of sums is compensated: two levels / compensated / pgemm_kernel 70B down
    // 1.77e-7 / 1.16e-7 / 1.29e-7, 8B down 1.38e-7 / 1.20e-7 / 1.21e-7, K = 4096 1.46e-7 / 1.07e-7 / 1.18e-7, in the same time
    // as long as four waves fit a SIMD (LM head of 128256 at 32 rows 192 us; with the lo products in sums of their own the
    // error is 0.7e-7, but three waves fit: 199 us).
    auto flush = [&]() {
#pragma unroll
        for (int i = 0; i < MTW; ++i)
#pragma unroll
            for (int ct = 0; ct < NC; ++ct) {
                if (COMP) {   // `lost`: what the last sum rounded away
                    const f32x4 add = acc[i][ct] - lost[i][ct], sum = total[i][ct] + add;
                    lost[i][ct] = (sum - total[i][ct]) - add;
                    total[i][ct] = sum;
                } else {
                    total[i][ct] += acc[i][ct];
                }
                acc[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
    };
    int it0 = 0;
    bool odd = false;
    for (; it0 + 2 * QDW <= n_iter; it0 += QDW) {
#pragma unroll
        for (int u = 0; u < QDW; ++u) ktile(u, it0 + u, true);
        if (TWO && (odd || !BLOCKS)) flush();
        odd = !odd;
    }
    for (; it0 < n_iter; it0 += QDW) {
#pragma unroll
        for (int u = 0; u < QDW; ++u) {
            const int it = it0 + u;
            if (it < n_iter) ktile(u, it, it + QDW < n_iter);
        }
    }
    if (TWO) {
#pragma unroll
        for (int i = 0; i < MTW; ++i)
#pragma unroll
            for (int ct = 0; ct < NC; ++ct) {
                if (COMP) acc[i][ct] -= lost[i][ct];
                acc[i][ct] += total[i][ct];
            }
    }

    // acc[i][ct][v] of lane l: row 16 * (half * MTW + i) + l%16, column 4*(l/16) + v of tile q_tile(c16 + ct)
    const int row0 = m_base + 16 * half * MTW, r = lane & 15, kg = lane >> 4;
    if constexpr (FORM == PARTS) {
#pragma unroll
        for (int ct = 0; ct < NC; ++ct) {
            if (c16 + ct >= NT16) continue;
            const int col = q_tile<false>(a, c16 + ct) * 16 + 4 * kg;
#pragma unroll
            for (int i = 0; i < MTW; ++i) {
                const int row = row0 + 16 * i + r;
                if (row < a.part_rows) *reinterpret_cast<f32x4 *>(a.partials + ((size_t)j * a.part_rows + row) * a.Ntot + col) = acc[i][ct];
            }
        }
        return;
    }
    const EpilogueArgs e = epilogue_arguments();
    // A unit is a wave's pair p of column tiles on row tile i: an epilogue unit (rotary partners, gate and up) or 32 columns.
    constexpr int NP = NC / 2, UW = MTW * NP;
    const int qkv_bits = e.d == 128 ? 2 : 1;   // QKV: rotary pairs of tiles per head, 4 or 2
    auto epilogue = [&](auto which) {   // one of them for all units, so that units overlap
        constexpr int EPI = decltype(which)::value;
        constexpr bool SCALED = EPI != FEPI_RESID && EPI != FEPI_STORE;
        auto inputs = [&](int i, int p) -> QuadIn {
            QuadIn in{};
            const int m = min(row0 + 16 * i + r, e.M - 1), t0 = c16 + 2 * p, unit = (c16 >> 1) + p;
            if (t0 >= NT16) return in;
            if (EPI == FEPI_RESID) {
                const int c0 = t0 * 16 + 4 * kg, c1 = t0 + 1 < NT16 ? c0 + 16 : c0;
                in.x0 = load4(e.X + (size_t)m * e.h + c0);
                in.x1 = load4(e.X + (size_t)m * e.h + c1);
                __builtin_memcpy(&in.g0, e.gamma_next + c0, 8);   // caller's array: no alignment assumed
                __builtin_memcpy(&in.g1, e.gamma_next + c1, 8);
            } else if (EPI == FEPI_QKV) {
                in.base = e.pos_base[e.by_k1(m)];
                if (unit >> qkv_bits < e.nq + e.nkv) {
                    const float *cs = e.rope_cs + ((size_t)e.rope_pos[m] * (e.d >> 1) + (unit & ((1 << qkv_bits) - 1)) * 16 + 4 * kg) * 2;
                    in.x0 = load4(cs);
                    in.x1 = load4(cs + 4);
                }
            }
            return in;
        };
        auto finish = [&](int i, int p, const f32x4 &v0, const f32x4 &v1, const QuadIn &in, float &ss, Best &best) {
            const int ml = 16 * (half * MTW + i) + r, m = m_base + ml, t0 = c16 + 2 * p, unit = (c16 >> 1) + p;
            if (m >= e.M || t0 >= NT16) return;
            const int c0 = t0 * 16 + 4 * kg;
            const bool two = t0 + 1 < NT16;
            if (EPI == FEPI_SWIGLU) {
                swiglu4(e, m, unit * 16 + 4 * kg, rstd_s[ml], v0, v1);
            } else if (EPI == FEPI_QKV) {
                qkv4(e, m, unit >> qkv_bits, (unit & ((1 << qkv_bits) - 1)) * 16 + 4 * kg, rstd_s[ml], v0, v1, in);
            } else if (EPI == FEPI_RESID) {
                ss += resid4(e, m, c0, v0, in.x0, in.g0);
                if (two) ss += resid4(e, m, c0 + 16, v1, in.x1, in.g1);
            } else if (EPI == FEPI_LM) {
                lm4(e, m, c0, rstd_s[ml], v0, best);
                if (two) lm4(e, m, c0 + 16, rstd_s[ml], v1, best);
            } else {
                *reinterpret_cast<f32x4 *>(e.out + (size_t)m * e.Ntot + c0) = v0;
                if (two) *reinterpret_cast<f32x4 *>(e.out + (size_t)m * e.Ntot + c0 + 16) = v1;
            }
        };
        if constexpr (FORM == WHOLE) {
            Best best[MTW];
#pragma unroll
            for (int i = 0; i < MTW; ++i) best[i] = Best::none();
            // Of the next unit: the compiler requests nothing ahead of a unit's stores, which might change it (tiny shape, 128 rows, where four
            // workgroups each finish eight units a wave: QKV 16.4 -> 15.3 us, O 13.2 -> 12.3).
            QuadIn ahead = inputs(0, 0);
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int i = 0; i < MTW; ++i) {
                    const QuadIn in = ahead;
                    if (i + 1 < MTW) ahead = inputs(i + 1, p);
                    else if (p + 1 < NP) ahead = inputs(0, p + 1);
                    float ss = 0.f;
                    finish(i, p, acc[i][2 * p], acc[i][2 * p + 1], in, ss, best[i]);
                    if (EPI == FEPI_RESID) {   // one sum of squares per row and pair
                        ss = row_sum4(ss);
                        const int m = row0 + 16 * i + r;
                        if (kg == 0 && m < e.M && c16 + 2 * p < NT16) e.ssq_out[(size_t)m * e.nss_out + (c16 >> 1) + p] = ss;
                    }
                }
            if (EPI == FEPI_LM) {   // one arg-max per row and workgroup
                __syncthreads();      // the ring has been read
                Best(*best_s)[16 * MT16] = reinterpret_cast<Best(*)[16 * MT16]>(lds);
#pragma unroll
                for (int i = 0; i < MTW; ++i) {
                    best[i].across(16);
                    best[i].across(32);
                    if (kg == 0) best_s[cg][16 * (half * MTW + i) + r] = best[i];
                }
                __syncthreads();
                for (int row = threadIdx.x; row < 16 * MT16; row += QW * 64) {
                    if (m_base + row >= e.M) continue;
                    Best all = best_s[0][row];
#pragma unroll
                    for (int x = 1; x < CW; ++x) all.take(best_s[x][row].v, best_s[x][row].i);
                    e.part_val[(size_t)(m_base + row) * e.n_part + grp] = all.v;
                    e.part_idx[(size_t)(m_base + row) * e.n_part + grp] = all.i;
                }
            }
            return;
        }
        if constexpr (FORM == DIE) {
            // Unit v = i * NP + p belongs to slice v modulo J.  The others' units are stored as the lanes hold them, its own stay in registers
            // until the other slices of them have arrived.
            constexpr int ROOM = BLOCKS ? 8 : UW;   // units a wave has room for (blocks of eight and six tiles mix)
            constexpr int SLICE = QW * ROOM * 2048; // bytes
            const int J = e.J;
            float *const slot = e.hand.parts + ((size_t)set * J + j) * (SLICE / 4) + wave * (ROOM * 512) + lane * 4;
            auto put = [&](bool own) {
                int o = 0;
#pragma unroll
                for (int v = 0; v < UW; ++v) {
                    if ((o == j) == own) {
                        *reinterpret_cast<f32x4 *>(slot + v * 512) = acc[v / NP][v % NP * 2];
                        *reinterpret_cast<f32x4 *>(slot + v * 512 + 256) = acc[v / NP][v % NP * 2 + 1];
                    }
                    if (++o == J) o = 0;
                }
            };
            put(false);
            const uint64_t seen = hand_arrive(e.hand, set);
            QuadIn in[2];
            in[0] = inputs(min(j, UW - 1) / NP, min(j, UW - 1) % NP);   // of the first two units of its share
            in[1] = inputs(min(j + J, UW - 1) / NP, min(j + J, UW - 1) % NP);
            if (SCALED) {
                scales.load(e.ssq_in, e.nss_in, e.M, m_base, 0);
                scales.finish(e, m_base, rstd_s);   // published by the barrier of hand_wait
            }
            int *way_s = reinterpret_cast<int *>(rstd_s + 16 * MT16);
            HandWay way = hand_wait(e.hand, set, J, seen, way_s);
            uint64_t left = way == HAND_SHARE ? hand_leave(e.hand, set) : 0;
            if (way == HAND_TURN_IN) {
                put(true);
                way = hand_turn_in(e.hand, set, J, way_s);
            }
            if (way != HAND_NOTHING) {
                const DieBuffer parts(e.hand.parts + (size_t)set * J * (SLICE / 4), (size_t)J * SLICE);
                const int at = wave * (ROOM * 2048) + lane * 16, first = way == HAND_ALL ? 0 : j, step = way == HAND_ALL ? 1 : J;
                float2 (*const row_s)[QW][16] = reinterpret_cast<float2 (*)[QW][16]>(lds);   // [unit of the share][wave][row]
                auto done = [&](int v, const f32x4 &v0, const f32x4 &v1, const QuadIn &u) {
                    float ss = 0.f;
                    Best best = Best::none();
                    finish(v / NP, v % NP, v0, v1, u, ss, best);
                    const int k = way == HAND_ALL ? v : e.by_J(v);
                    if (EPI == FEPI_RESID) {
                        ss = row_sum4(ss);
                        if (kg == 0) row_s[k][wave][r] = float2{ss, 0.f};
                    } else if (EPI == FEPI_LM) {
                        best.across(16);
                        best.across(32);
                        if (kg == 0) row_s[k][wave][r] = float2{best.v, __int_as_float(best.i)};
                    }
                };
                // U units of the share from v0 on, up to N other slices of each in flight, added in the order of the slices (equal columns keep equal sums).
                auto share = [&](auto units, auto slices, int v0) {
                    constexpr int U = decltype(units)::value, N = decltype(slices)::value;
                    f32x4 own[U][2], sum[U][2], t[U][N][2];
                    auto unit = [&](int k) { return min(v0 + k * step, UW - 1); };   // past the last: not used
                    auto request = [&](int n0) {
#pragma unroll
                        for (int k = 0; k < U; ++k)
                            if (k == 0 || v0 + k * step < UW)
#pragma unroll
                                for (int n = 0; n < N; ++n)
                                    if (n0 + n < J - 1) {
                                        const int v = unit(k), o = way == HAND_ALL ? v - e.by_J(v) * J : j, q = n0 + n + (n0 + n >= o);
                                        t[k][n][0] = parts.load4(at, q * SLICE + v * 2048);
                                        t[k][n][1] = parts.load4(at, q * SLICE + v * 2048 + 1024);
                                    }
                    };
                    request(0);
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        const int mine = unit(k);
                        sum[k][0] = sum[k][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                        if (way == HAND_ALL) {
                            const int o = mine - e.by_J(mine) * J;
                            own[k][0] = parts.load4(at, o * SLICE + mine * 2048);
                            own[k][1] = parts.load4(at, o * SLICE + mine * 2048 + 1024);
                        } else {
#pragma unroll
                            for (int v = 0; v < UW; ++v)
                                if (v == mine) {
                                    own[k][0] = acc[v / NP][v % NP * 2];
                                    own[k][1] = acc[v / NP][v % NP * 2 + 1];
                                }
                        }
                    }
                    for (int n0 = 0; n0 < J - 1; n0 += N) {
                        if (n0 > 0) request(n0);
#pragma unroll
                        for (int k = 0; k < U; ++k)
#pragma unroll
                            for (int n = 0; n < N; ++n) {
                                const int v = unit(k), o = way == HAND_ALL ? v - e.by_J(v) * J : j;
                                if (n0 + n < J - 1) {
                                    if (n0 + n == o) {
                                        sum[k][0] += own[k][0];
                                        sum[k][1] += own[k][1];
                                    }
                                    sum[k][0] += t[k][n][0];
                                    sum[k][1] += t[k][n][1];
                                }
                            }
                    }
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if ((way == HAND_ALL ? unit(k) - e.by_J(unit(k)) * J : j) == J - 1) {
                            sum[k][0] += own[k][0];
                            sum[k][1] += own[k][1];
                        }
                    if constexpr (U <= 2) {
#pragma unroll
                        for (int k = 0; k < U; ++k)
                            if (v0 + k * step < UW) {
                                if (way == HAND_ALL || v0 != j) in[k] = inputs(unit(k) / NP, unit(k) % NP);
                                done(unit(k), sum[k][0], sum[k][1], in[k]);
                            }
                    } else {
                        for (int k = 0; k < U && v0 + k * step < UW; ++k) {
                            f32x4 s0 = sum[0][0], s1 = sum[0][1];
#pragma unroll
                            for (int x = 1; x < U; ++x)
                                if (x == k) { s0 = sum[x][0]; s1 = sum[x][1]; }
                            done(unit(k), s0, s1, inputs(unit(k) / NP, unit(k) % NP));
                        }
                    }
                };
                constexpr int N = QW == 8 ? 4 : 8;
                if (J == 2) {
                    constexpr int U = (UW + 1) / 2 > 2 ? (UW + 1) / 2 : 2;
                    for (int v0 = first; v0 < UW; v0 += U * step) share(std::integral_constant<int, U>{}, std::integral_constant<int, 1>{}, v0);
                } else {
                    for (int v0 = first; v0 < UW; v0 += 2 * step) share(std::integral_constant<int, 2>{}, std::integral_constant<int, N>{}, v0);
                }
                if (EPI == FEPI_RESID || EPI == FEPI_LM) {   // one sum of squares or maximum per row, group and pair of column tiles
                    __syncthreads();
                    const int n_units = first < UW ? e.by_J(UW - 1 - first) + 1 : 0, count = way == HAND_ALL ? UW : n_units;
                    for (int x = threadIdx.x; x < count * 16 * RH; x += QW * 64) {
                        const int k = x / (16 * RH), h = x / 16 % RH, v = first + k * step, m = m_base + 16 * (h * MTW + v / NP) + (x & 15);
                        const int per_row = EPI == FEPI_LM ? e.n_part : e.nss_out, place = grp * NP + v % NP;
                        if (m >= e.M || place >= per_row) continue;   // the second pair where there is only one
                        const size_t to = (size_t)m * per_row + place;
                        float2 all = row_s[k][h * CW][x & 15];
                        if (EPI == FEPI_LM) {
                            Best best{all.x, __float_as_int(all.y)};
#pragma unroll
                            for (int w2 = 1; w2 < CW; ++w2) best.take(row_s[k][h * CW + w2][x & 15].x, __float_as_int(row_s[k][h * CW + w2][x & 15].y));
                            e.part_val[to] = best.v;
                            e.part_idx[to] = best.i;
                        } else {
#pragma unroll
                            for (int w2 = 1; w2 < CW; ++w2) all.x += row_s[k][h * CW + w2][x & 15].x;
                            e.ssq_out[to] = all.x;
                        }
                    }
                }
            }
            if (way != HAND_SHARE) left = hand_leave(e.hand, set);
            hand_clear(e.hand, set, J, left);
        }
    };
    switch (e.epi) {
    case FEPI_QKV: epilogue(std::integral_constant<int, FEPI_QKV>{}); break;
    case FEPI_RESID: epilogue(std::integral_constant<int, FEPI_RESID>{}); break;
    case FEPI_SWIGLU: epilogue(std::integral_constant<int, FEPI_SWIGLU>{}); break;
    case FEPI_LM: epilogue(std::integral_constant<int, FEPI_LM>{}); break;
    default:
        if constexpr (FORM == WHOLE) epilogue(std::integral_constant<int, FEPI_STORE>{});   // kernel-level GEMMs do not hand over
        break;
    }
}

// BLOCKS: RB blocks of rows, of MT16 tiles, or (MT16 = 0) the first n8 of eight tiles and the others of six.  Blocks of one
// size have kernels of their own: in the mixed one they are 2 % slower.
template <int MT16, int QW, bool BLOCKS, int FORM>
// Registers: two workgroups of four waves per compute unit up to nine tiles (tiny shape with a vocabulary of 128256, a step of 144 rows:
// 324 registers and one workgroup 138 us, 256, six of them spilled, and two 116), which at three tiles costs more than it gives (8B
// gate/up at 33 rows 44.4 -> 45.2); four waves per SIMD up to two tiles; summed inside the launch one workgroup, which is all it has.
__global__ __launch_bounds__(QW * 64) __attribute__((amdgpu_waves_per_eu(FORM == DIE ? 1 : (!BLOCKS && MT16 <= 2 ? 4 : (QW == 4 && MT16 >= 4 && MT16 <= 9 ? 2 : 1))))) void qgemm16_kernel(FusedGemmArgs a, int RB, int n8, int NT16, int pairs)
{
    constexpr int MOST = MT16 ? MT16 : 8;   // row tiles of a workgroup at most
    __shared__ u32x4 lds[QShape<MOST, QW, BLOCKS, FORM>::LDS];
    __shared__ float rstd_s[FORM == PARTS ? 1 : 16 * MOST + 1];   // ... and a word for the hand-over
    const int bid = blockIdx.x;
    int rb = 0, grp, j, set = 0;
    if constexpr (FORM == DIE) {   // `pairs` column groups; on each die every eighth of them, with its slices and their row blocks side by side
        const int slot = bid >> 3, x = BLOCKS ? a.by_RB(slot) : slot, local = a.by_J(x);
        rb = slot - x * (BLOCKS ? RB : 1);
        j = x - local * a.J;
        grp = local * 8 + (bid & 7);
        if (grp >= pairs) return;
        set = grp * (BLOCKS ? RB : 1) + rb;
    } else {
        int gj = bid;
        if constexpr (BLOCKS) {
            const int whole = pairs & ~7;   // (column group, slice) pairs; those in full sets of 8
            const bool in_set = bid < whole * RB;
            const int x = in_set ? bid >> 3 : bid - whole * RB, by = in_set ? RB : pairs - whole;
            const int q = (int)((unsigned)x / (unsigned)by), r = x - q * by;
            rb = in_set ? r : q;
            gj = in_set ? q * 8 + (bid & 7) : whole + r;
        }
        // WHOLE: J is 1, but a value of the launch all the same.  With a k-range known to begin at zero the addresses of the loads in
        // flight take 8-24 registers more (17..32 rows: spills, 1.03 x the time).
        grp = (int)((unsigned)gj / (unsigned)a.J);
        j = gj - grp * a.J;
    }
    if constexpr (!BLOCKS) qgemm16_rows<MT16, QW, false, FORM>(a, NT16, 0, grp, j, set, lds, rstd_s);
    else if constexpr (MT16 != 0) qgemm16_rows<MT16, QW, true, FORM>(a, NT16, MT16 * rb, grp, j, set, lds, rstd_s);
    else if (rb < n8) qgemm16_rows<8, QW, true, FORM>(a, NT16, 8 * rb, grp, j, set, lds, rstd_s);
    else qgemm16_rows<6, QW, true, FORM>(a, NT16, 8 * n8 + 6 * (rb - n8), grp, j, set, lds, rstd_s);
}

// Row blocks of a launch: one of up to ten tiles, more of eight (the sums in two levels leave no registers for more), as many
// of them of six as the rows allow: 20 tiles are 8 + 6 + 6, not three of eight.  Three of eight / 8 + 6 + 6 / two passes of
// ten with sums in one level, us: 320 rows 8B gate/up 180 / 171 / 164, 70B gate/up 618 / 582 / 563, down 312 / 291 / 298; 400
// rows (four of eight / 8 + 6 + 6 + 6) 70B gate/up 794 / 744 / 732, LM head of 128256 924 / 850 / 906.
struct RowBlocks {
    int RB, n8;   // blocks, those of eight tiles
};
__host__ RowBlocks row_blocks(int mt16)
{
    if (mt16 <= 10) return RowBlocks{1, 0};
    const int RB = (mt16 + 7) / 8, spare = (8 * RB - mt16) / 2;
    return RowBlocks{RB, RB - (spare < RB ? spare : RB)};
}

struct QPlan {
    int groups, J, kps;   // column groups, K slices (none empty), k-tiles per slice
    int qw;               // waves (32-column tiles) per workgroup
};

// Column groups and the K split.  The split is the smallest J whose groups*J workgroups fill whole
// rounds of one workgroup per compute unit to at least 85 % (else the best-filling one), with at least
// 8 k-tiles per slice and at most 16 slices.  More slices than that would still find room on the device at
// up to 96 rows (two workgroups fit a compute unit there), but every slice is another fp32 copy of the
// output to write and read back: measured on the 70B shapes at 80 rows, filling 256 slots instead of 512
// took QKV from 52 to 43 us, down from 113 to 91 us, O from 46 to 41 us.
__host__ QPlan q_plan(int Ntot, int K, int M)
{
    const int NT32 = (Ntot / 16 + 1) / 2, KT = (K + 31) / 32;
    const int mt32 = M >= 160 ? 5 : (M + 31) / 32;
    const size_t bytes = (size_t)Ntot * (size_t)K * 2;
    QPlan p;
    // Four waves (128 columns per workgroup, K split half as often): the small matrices, and every matrix but
    // the very large ones at up to 64 rows (measured at 36 and 64 rows on the 8B shapes: gate/up 59 -> 48 and
    // 64 -> 51 us, down 34 -> 32 and 37 -> 33 us; from 65 rows on eight waves win on the large matrices, and
    // on the 940 MB gate/up matrix of the 70B shape they win at 48 rows already: 189 -> 153 us without a split).
    p.qw = (bytes < ((size_t)64 << 20) || (mt32 <= 2 && bytes < ((size_t)512 << 20))) ? 4 : 8;
    const int slots = 256;
    p.groups = (NT32 + p.qw - 1) / p.qw;
    int jmax = KT / 8;
    if (jmax > 16) jmax = 16;
    if (jmax < 1) jmax = 1;
    int best = 1;
    double best_fill = 0.0;
    for (int J = 1; J <= jmax; ++J) {
        const long tasks = (long)p.groups * J;
        const long rounds = (tasks + slots - 1) / slots;
        const double fill = (double)tasks / (double)(rounds * slots);
        if (fill > best_fill + 1e-9) { best_fill = fill; best = J; }
        if (fill >= 0.85) { best = J; break; }
    }
    if (M > 160) {
        // Row blocks fill the device as well as slices do, without partial sums: the split with the least estimated time
        //   rounds x (k-tiles per slice x row tiles x 0.099 us + 10.6 us) + 0.13 us per MB of partial sums to read back,
        // fitted to the 8B shapes at 256 and 512 rows, eight waves throughout.  Measured there, GEMM and epilogue launch at
        // 512 rows, J = 1 / 2 / 3 / 4 / 6 / 8: QKV 103 / 66 / 95 / 75 / 88 / 82 us, O 100 / 61 / 50 / 45 / 61 / 58, gate/up
        // 290 / 301 / 315 / 324 / 385 / 451, down 322 / 174 / 133 / 109 / 142 / 122 (four passes of up to 160 rows took 126,
        // 101, 294 + 30 and 190 + 19 us).  No split needs more than SPLIT_BYTES of partial sums unless the rule above did.
        constexpr size_t SPLIT_BYTES = (size_t)32 << 20;
        const int was = best, mt16 = (M + 15) / 16;
        const RowBlocks rows = row_blocks(mt16);
        const int RB = rows.RB;
        const double mt = (8.0 * rows.n8 + 6.0 * (RB - rows.n8)) / RB;
        p.qw = 8;
        p.groups = (NT32 + p.qw - 1) / p.qw;
        double least = 0.0;
        for (int J = 1; J <= jmax; ++J) {
            const size_t sums = (size_t)J * mt16 * 16 * Ntot * sizeof(float);
            if (J > was && sums > SPLIT_BYTES) break;
            const long tasks = (long)p.groups * RB * J, rounds = (tasks + slots - 1) / slots;
            const double us = (double)rounds * ((KT + J - 1) / J * mt * 0.099 + 10.6) + 0.13e-6 * (double)sums;
            if (J == 1 || us < least) { least = us; best = J; }
        }
    }
    p.kps = (KT + best - 1) / best;
    p.J = (KT + p.kps - 1) / p.kps;
    return p;
}

// Which kernel a GEMM takes: true for pgemm_kernel.
//   17..32 rows: pgemm_kernel feeds every compute unit twice the weight bytes it would stream alone, which costs more than
//   the partial sums of qgemm16_kernel on all but the small matrices.  At 32 rows, GEMM and epilogue, pgemm / qgemm16 us:
//   8B QKV (50 MB) 14.8 / 16.0, O (34 MB) 11.4 / 14.3, down (117 MB) 30 / 26, gate/up (235 MB) 50 / 42, LM head 223 / 193,
//   70B QKV (168 MB) 41 / 32, gate/up 206 / 143, down 107 / 76.  The line lies between the 50 MB and the 117 MB of these.
//   1..16 rows: pgemm_kernel wins wherever a workgroup covers the whole K (4096); where K is split, its slices go through
//   memory too, and from 256 MB the faster stream decides, pgemm / qgemm16 at 16 rows: 70B gate/up (940 MB) 150 / 142,
//   down (470 MB) 79 / 73, QKV (168 MB) 32 / 32, O (134 MB) 26 / 30, and an 8B layer with its down projection
//   (117 MB) on qgemm16 108.1 -> 109.7 us.
// A GEMM whose partial sums would exceed SMALL_SCRATCH (the library's own array for callers without scratch) stays.
__host__ bool is_small(int M, int Ntot, int K)
{
    constexpr size_t SMALL_SCRATCH = (size_t)32 << 20;
    if (M > 32) return false;
    const size_t bytes = (size_t)Ntot * (size_t)K * 2;
    if (M > 16 ? bytes < ((size_t)64 << 20) : K <= PW * 8 * 32 || bytes < ((size_t)256 << 20)) return true;
    return (size_t)q_plan(Ntot, K, M).J * round_up(M, 16) * Ntot * sizeof(float) > SMALL_SCRATCH;
}

// The same split for slices that are summed inside the launch: one workgroup per compute unit (they wait for each other), the slices of
// a column group on one die.  False, and the plan as it was, where that leaves no split.
// As many slices as a die has compute units for (one row block): what a slice costs here is a share of one die's L2, not a copy of the
// output in memory.  With row blocks no more than the plan above: they fill the device already.
// Against partial sums and an epilogue launch, us a step: 70B layer at 144 rows 588 -> 570; two 8B layers at 36 rows 443 -> 428, 160 rows
// 558 -> 544, 512 rows 968 -> 950; layer and head at 91 rows 402 -> 394.
//
// Row blocks and a number of column groups that eight dies cannot share evenly leave dies with fewer workgroups, and fewer slices
// than the plan above: not where the k-tiles that every workgroup then has more cost more (0.099 us a row tile, as in q_plan) than an epilogue
// launch and its partial sums (5 us and 0.13 us per MB).  18944 x 3584 at 300 rows, 14 groups, five slices instead of six: 94.5 us inside
// the launch, 77.4 and 9.2 with partial sums; 3584 x 4608, 18 groups, three instead of four: 42.1, 28.1 and 12.4.
// Steps of two layers at 512 rows without / with this line, us: hidden 5120, FFN 13824 1208 / 1143; 3072, 24576 1075 / 1032; 4608, 18432
// 1482 / 1401; 2560, 9728 644 / 621.
__host__ bool die_plan(QPlan &p, int KT, const RowBlocks &rows, size_t slice_bytes)
{
    const int RB = rows.RB;
    const int per_die = (p.groups + 7) / 8 * RB;   // workgroups of a die for one slice
    int J = 32 / per_die;
    if (J > KT / 8) J = KT / 8;
    if (J > 16) J = 16;
    if (RB > 1 && J > p.J) J = p.J;
    if (J < 2 || round_up(p.groups, 8) * RB > HAND_GROUPS) return false;
    const int kps = (KT + J - 1) / J;
    if (RB > 1 && (kps - p.kps) * ((8.0 * rows.n8 + 6.0 * (RB - rows.n8)) / RB) * 0.099 > 5.0 + 0.13e-6 * (double)slice_bytes * p.J) return false;
    p.kps = kps;
    p.J = (KT + p.kps - 1) / p.kps;
    return true;
}

struct LargePlan {
    QPlan p;
    RowBlocks rows;
    bool die;            // slices summed inside the launch
    int sums, maxima;    // values per row: RESID sums of squares, LM arg-max partials
    size_t hand_bytes;   // of Hand's parts
};

// `hand`: the launch has words for a hand-over.  Summed inside the launch every group of columns leaves a value per pair of tiles that its
// waves hold, two with row blocks -- but no more than there are pairs: one column tile is one pair, and the buffers behind the values
// have room for one per 16 columns.
__host__ LargePlan large_plan(int Ntot, int KT, int M, bool hand)
{
    const int mt16 = (M + 15) / 16, pairs = (Ntot / 16 + 1) / 2;
    LargePlan l;
    l.p = q_plan(Ntot, KT * 32, M);
    l.rows = row_blocks(mt16);
    l.die = hand && l.p.J > 1 && die_plan(l.p, KT, l.rows, (size_t)mt16 * 16 * Ntot * sizeof(float));
    const int values = l.p.groups * (l.rows.RB > 1 ? 2 : 1);
    l.sums = l.die && values < pairs ? values : pairs;
    l.maxima = l.die ? l.sums : l.p.groups;
    const int units = l.rows.RB > 1 ? 8 : (mt16 < 2 ? 2 : mt16);   // a wave has room for
    l.hand_bytes = l.die ? (size_t)l.p.groups * l.rows.RB * l.p.J * l.p.qw * units * 2048 : 0;
    return l;
}

template <int EPI> hipError_t launch_large(FusedGemmArgs &a, hipStream_t s, bool *needs_epilogue, hipEvent_t t0, hipEvent_t t1)
{
    const int NT16 = a.Ntot / 16;
    const LargePlan plan = large_plan(a.Ntot, a.KT, a.M, a.hand.words != nullptr);
    const QPlan &p = plan.p;
    const int mt16 = (a.M + 15) / 16;
    const RowBlocks &rows = plan.rows;
    const bool die = plan.die;
    a.J = p.J;
    a.kps = p.kps;
    a.by_J = Div(p.J);
    a.by_RB = Div(rows.RB);
    a.part_rows = round_up(a.M, 16);
    a.epi = EPI;
    a.nss_out = plan.sums;   // read where this launch leaves them (RESID)
    a.n_part = plan.maxima;
    *needs_epilogue = a.J > 1 && !die;   // an unsplit K: the kernel applies the epilogue itself
    if (plan.hand_bytes > HAND_PARTS) return hipErrorInvalidValue;
    if (EPI == FEPI_QKV) { a.seg0 = a.nq * (a.d >> 4); a.seg1 = a.nkv * (a.d >> 4); }
    else if (EPI == FEPI_SWIGLU) { a.seg0 = a.NT; a.seg1 = a.NT; }
    else { a.seg0 = NT16; a.seg1 = 0; }
    if (*needs_epilogue && (size_t)a.J * a.part_rows * a.Ntot * sizeof(float) > a.partial_bytes) return hipErrorInvalidValue;
    const dim3 grid((die ? round_up(p.groups, 8) : p.groups) * a.J * rows.RB), block(p.qw * 64);
#define SSSD_Q16LAUNCH(MT, QW, BLOCKS)                                                                                                          \
    do {                                                                                                                                        \
        if (die) hipExtLaunchKernelGGL((qgemm16_kernel<MT, QW, BLOCKS, DIE>), grid, block, 0, s, t0, t1, 0, a, rows.RB, rows.n8, NT16, p.groups); \
        else if (a.J == 1) hipExtLaunchKernelGGL((qgemm16_kernel<MT, QW, BLOCKS, WHOLE>), grid, block, 0, s, t0, t1, 0, a, rows.RB, rows.n8, NT16, p.groups); \
        else hipExtLaunchKernelGGL((qgemm16_kernel<MT, QW, BLOCKS, PARTS>), grid, block, 0, s, t0, t1, 0, a, rows.RB, rows.n8, NT16, p.groups * a.J);   \
    } while (0)
#define SSSD_Q16ROWS(MT)                                  \
    do {                                                  \
        if (p.qw == 8) SSSD_Q16LAUNCH(MT, 8, false);      \
        else SSSD_Q16LAUNCH(MT, 4, false);                \
    } while (0)
    if (rows.RB > 1) {
        if (rows.n8 == 0) SSSD_Q16LAUNCH(6, 8, true);
        else if (rows.n8 == rows.RB) SSSD_Q16LAUNCH(8, 8, true);
        else SSSD_Q16LAUNCH(0, 8, true);
    } else {
        switch (mt16) {
        case 1:   // the second row tile is padding, computed and not stored
        case 2: SSSD_Q16ROWS(2); break;
        case 3: SSSD_Q16ROWS(3); break;
        case 4: SSSD_Q16ROWS(4); break;
        case 5: SSSD_Q16ROWS(5); break;
        case 6: SSSD_Q16ROWS(6); break;
        case 7: SSSD_Q16ROWS(7); break;
        case 8: SSSD_Q16ROWS(8); break;
        case 9: SSSD_Q16ROWS(9); break;
        default: SSSD_Q16ROWS(10); break;
        }
    }
#undef SSSD_Q16ROWS
#undef SSSD_Q16LAUNCH
    return hipGetLastError();
}

// k-tiles per wave: as many as share a short K out over the 16 waves -- with eight, the waves past the end of a K of 256 fetched
// eight tiles of padding each, and a launch was bound by them (tiny model, five rows: 62.3 -> 55.2 us a step) -- else 7 when K is a multiple of
// 16*7*32 but not of 16*8*32 (the FFN widths of the Llama shapes), else 8.  A ragged K split is legal in every case.
__host__ int small_kpw(int KT)
{
    if (KT <= PW * 4) return KT <= PW ? 1 : (KT <= PW * 2 ? 2 : 4);
    return (KT % (PW * 7) == 0 && KT % (PW * 8) != 0) ? 7 : 8;
}

struct SmallPlan {
    int rh, kpw, J, upw, groups;
};

__host__ SmallPlan small_plan(const FusedGemmArgs &a)
{
    SmallPlan p;
    p.rh = a.M > 16 ? 2 : 1;   // 17..32 rows: every workgroup twice, one per row tile
    p.kpw = small_kpw(a.KT);
    p.J = (a.KT + PW * p.kpw - 1) / (PW * p.kpw);
    const int n_cu = (a.n_cu > 0 ? a.n_cu : 256) / p.rh;
    int groups_target = n_cu / p.J;
    if (groups_target < 1) groups_target = 1;
    p.upw = (a.n_units + groups_target - 1) / groups_target;
    p.groups = (a.n_units + p.upw - 1) / p.upw;
    return p;
}

template <int EPI> hipError_t launch_small(FusedGemmArgs &a, hipStream_t s, bool *needs_epilogue, hipEvent_t t0, hipEvent_t t1)
{
    const SmallPlan sp = small_plan(a);
    const int kpw = sp.kpw, groups = sp.groups;
    a.J = sp.J;
    a.upw = sp.upw;
    a.groups = sp.groups;
    a.part_rows = 16 * sp.rh;
    a.nss_out = a.h >> 4;
    a.n_part = sp.groups;
    if (a.J > 1 && (size_t)a.J * a.part_rows * a.Ntot * sizeof(float) > a.partial_bytes) return hipErrorInvalidValue;
    if (EPI != FEPI_RESID && EPI != FEPI_STORE && a.J == 1 && a.nss_in > small_row_sums(kpw)) return hipErrorInvalidValue;
    const dim3 grid(groups * a.J * sp.rh), block(PW * 64);
    if (groups * sp.rh > a.tail_slots) a.tail_count = nullptr;   // no counter for every group: epilogue launch
    const bool one = Unit<EPI>::TILES == 1 && a.upw == 1;   // one tile per workgroup
#define SSSD_PKERNEL(KPW, SPLIT, RH)                                                                                                       \
    do {                                                                                                                                   \
        if (one) hipExtLaunchKernelGGL((pgemm_kernel<EPI, KPW, SPLIT, RH, Unit<EPI>::TILES == 1>), grid, block, 0, s, t0, t1, 0, a);       \
        else hipExtLaunchKernelGGL((pgemm_kernel<EPI, KPW, SPLIT, RH, false>), grid, block, 0, s, t0, t1, 0, a);                           \
    } while (0)
#define SSSD_PLAUNCH(KPW, RH)                         \
    do {                                              \
        if (a.J > 1) SSSD_PKERNEL(KPW, true, RH);     \
        else SSSD_PKERNEL(KPW, false, RH);            \
    } while (0)
#define SSSD_PWHOLE(KPW)                              \
    do {                                              \
        if (sp.rh == 2) SSSD_PKERNEL(KPW, false, 2);  \
        else SSSD_PKERNEL(KPW, false, 1);             \
    } while (0)
    if (kpw == 1) SSSD_PWHOLE(1);
    else if (kpw == 2) SSSD_PWHOLE(2);
    else if (kpw == 4) SSSD_PWHOLE(4);
    else if (sp.rh == 2 && kpw == 7) SSSD_PLAUNCH(7, 2);
    else if (sp.rh == 2) SSSD_PLAUNCH(8, 2);
    else if (kpw == 7) SSSD_PLAUNCH(7, 1);
    else SSSD_PLAUNCH(8, 1);
#undef SSSD_PWHOLE
#undef SSSD_PLAUNCH
#undef SSSD_PKERNEL
    *needs_epilogue = a.J > 1 && !a.tail_count;
    return hipGetLastError();
}

}  // namespace

int stream_gemm_max_rows() { return 32; }

const char *stream_gemm_kernel_name(int M, int N, int K)
{
    return is_small(M, N, (K + 31) / 32 * 32) ? "pgemm_kernel" : "qgemm16_kernel";
}

// K slices of a GEMM of M rows, and the rows that each of its slices has in the split-K scratch.
static int gemm_slices(int M, int N, int K, int *rows)
{
    const int KT = (K + 31) / 32;
    if (!is_small(M, N, KT * 32)) {
        *rows = round_up(M, 16);
        return q_plan(N, KT * 32, M).J;
    }
    *rows = M <= 16 ? 16 : 32;
    const int ks = PW * small_kpw(KT);
    return (KT + ks - 1) / ks;
}

// Split-K scratch that a launch of M rows uses: none where the K is whole.
size_t stream_gemm_launch_bytes(int M, int N, int K)
{
    int rows;
    const size_t J = (size_t)gemm_slices(M, N, K, &rows);
    return J > 1 ? J * rows * N * sizeof(float) : 0;
}

// ... that any step of up to M rows uses: the K split depends on the number of row tiles, so the worst case over every size.
size_t stream_gemm_partial_bytes(const Dims &D, int M)
{
    size_t most = 0;
    auto consider = [&](int rows, int N, int K) {
        const size_t need = stream_gemm_launch_bytes(rows, N, K);
        if (need > most) most = need;
    };
    for (int rows = 16; rows <= round_up(M, 16); rows += 16) {
        consider(rows, D.qd + 2 * D.kd, D.h);
        consider(rows, D.h, D.qd);
        consider(rows, 2 * D.f, D.h);
        consider(rows, D.h, D.f);
        consider(rows, D.V, D.h);
    }
    return most;
}

// Values per row that a GEMM of M rows leaves at most, whichever form it takes: sums of squares (RESID) or arg-max partials (LM).
int stream_gemm_row_values(int M, int N, int K, bool lm)
{
    const int KT = (K + 31) / 32;
    if (is_small(M, N, KT * 32)) return N / 16;
    int most = 0;
    for (bool hand : {false, true}) {
        const LargePlan l = large_plan(N, KT, M, hand);
        const int epi_blocks = l.p.J > 1 && !l.die ? ((N + 31) / 32 + 3) / 4 : 0;   // epi_kernel's: four column blocks per workgroup at least
        for (int n : {epi_blocks, lm ? l.maxima : l.sums})
            if (n > most) most = n;
    }
    return most;
}

// Whether a GEMM of M rows, in a launch that has words for it, sums its slices inside the launch; room for what its workgroups hand over.
bool stream_gemm_hands_over(int M, int N, int K)
{
    const int KT = (K + 31) / 32;
    return !is_small(M, N, KT * 32) && large_plan(N, KT, M, true).die;
}

size_t stream_gemm_hand_bytes(int M, int N, int K)
{
    const int KT = (K + 31) / 32;
    return is_small(M, N, KT * 32) ? 0 : large_plan(N, KT, M, true).hand_bytes;
}

// What the kernel-level entry points ask for.  qgemm16_kernel applies the epilogue of a whole K itself and touches no scratch, but one
// copy of the output is asked for all the same: callers hold these sizes, and the entry point with scratch of its own refuses by them.
size_t stream_gemm_scratch_bytes(int M, int N, int K)
{
    int rows;
    const size_t J = (size_t)gemm_slices(M, N, K, &rows);
    return J > 1 || !is_small(M, N, (K + 31) / 32 * 32) ? J * rows * N * sizeof(float) : 0;
}

hipError_t launch_stream_gemm(FusedGemmArgs &a, int epilogue, hipStream_t s, bool *needs_epilogue, hipEvent_t t0,
                              hipEvent_t t1)
{
    if (epilogue == FEPI_QKV) {
        a.by_k1 = Div(a.k + 1);
        a.by_g = Div(a.nq / a.nkv);
    }
    if (!is_small(a.M, a.Ntot, a.KT * 32)) {
        switch (epilogue) {
        case FEPI_QKV: return launch_large<FEPI_QKV>(a, s, needs_epilogue, t0, t1);
        case FEPI_RESID: return launch_large<FEPI_RESID>(a, s, needs_epilogue, t0, t1);
        case FEPI_SWIGLU: return launch_large<FEPI_SWIGLU>(a, s, needs_epilogue, t0, t1);
        case FEPI_STORE: return launch_large<FEPI_STORE>(a, s, needs_epilogue, t0, t1);
        default: return launch_large<FEPI_LM>(a, s, needs_epilogue, t0, t1);
        }
    }
    switch (epilogue) {
    case FEPI_QKV: return launch_small<FEPI_QKV>(a, s, needs_epilogue, t0, t1);
    case FEPI_RESID: return launch_small<FEPI_RESID>(a, s, needs_epilogue, t0, t1);
    case FEPI_SWIGLU: return launch_small<FEPI_SWIGLU>(a, s, needs_epilogue, t0, t1);
    case FEPI_STORE: return launch_small<FEPI_STORE>(a, s, needs_epilogue, t0, t1);
    default: return launch_small<FEPI_LM>(a, s, needs_epilogue, t0, t1);
    }
}

hipError_t launch_stream_epilogue(FusedGemmArgs &a, int epilogue, hipStream_t s)
{
    switch (epilogue) {
    case FEPI_QKV: return launch_epi<FEPI_QKV>(a, s);
    case FEPI_RESID: return launch_epi<FEPI_RESID>(a, s);
    case FEPI_SWIGLU: return launch_epi<FEPI_SWIGLU>(a, s);
    case FEPI_STORE: return launch_epi<FEPI_STORE>(a, s);
    default: return launch_epi<FEPI_LM>(a, s);
    }
}
