// Device helpers of the weight-streaming GEMM kernels (stream_gemm.hip): MFMA wrapper, tile addressing
// of the concatenated outputs, device-scope accesses, the fused epilogues and the split-K slice sums.
#pragma once
#include "kernels.h"

namespace {

__device__ __forceinline__ f32x4 mfma(const u32x4 &a, const u32x4 &b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// A "unit" is what one epilogue invocation needs: a rotary tile pair (QKV), a gate tile and its
// up tile (SWIGLU), or a single tile.
template <int EPI> struct Unit {
    static constexpr int TILES = (EPI == FEPI_QKV || EPI == FEPI_SWIGLU) ? 2 : 1;
};

// Tile index of (unit, part) in the concatenated output [Q | K | V] or [gate | up].
template <int EPI> __device__ __forceinline__ int unit_tile(const FusedGemmArgs &a, int unit, int part)
{
    if (EPI == FEPI_QKV) {
        const int TH = a.d >> 4, per_head = TH >> 1;
        return (unit / per_head) * TH + unit % per_head + part * per_head;
    }
    if (EPI == FEPI_SWIGLU) return unit + part * a.NT;
    return unit;
}

// Packed weights of concatenated tile gt (k-tile 0, lane record 0).
template <int EPI> __device__ __forceinline__ const u32x4 *tile_weights(const FusedGemmArgs &a, int gt)
{
    const size_t stride = (size_t)a.KT * 64;
    if (EPI == FEPI_QKV) {
        const int TH = a.d >> 4, nqT = a.nq * TH, nkT = a.nkv * TH;
        if (gt < nqT) return a.W0 + gt * stride;
        if (gt < nqT + nkT) return a.W1 + (gt - nqT) * stride;
        return a.W2 + (gt - nqT - nkT) * stride;
    }
    if (EPI == FEPI_SWIGLU) return gt < a.NT ? a.W0 + gt * stride : a.W1 + (gt - a.NT) * stride;
    return a.W0 + gt * stride;
}

// Device-scope accesses (COH) for data that a workgroup of the SAME launch on another die wrote or
// will read: stores go through to memory, loads do not take a line this die cached earlier.  Plain
// accesses are enough across launches.
template <bool COH, typename T> __device__ __forceinline__ void st(T *p, T v)
{
    if (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

template <bool COH, typename T> __device__ __forceinline__ T ld(const T *p)
{
    if (COH) return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return *p;
}

// RESID, one element: row m, column n = unit * 16 + c, with what was read of the residual stream and the gains.  The 16 lanes of a row
// are adjacent.
template <bool COH>
__device__ __forceinline__ void resid1(const FusedGemmArgs &a, int unit, int m, int c, bool valid, float v0, float x, uint16_t gamma)
{
    const int n = unit * 16 + c;
    float xn = 0.f;
    if (valid) {
        xn = x + v0;
        st<COH>(a.X + (size_t)m * a.h + n, xn);
        uint16_t hi, lo;
        split_bf16(xn * bf16_to_f32(gamma), hi, lo);
        const size_t idx = packed_index(m, n, (a.h + 31) >> 5);
        st<COH>(a.out_hi + idx, hi);
        st<COH>(a.out_lo + idx, lo);
    }
    float ss = xn * xn;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 16);
    if (valid && c == 0) st<COH>(a.ssq_out + (size_t)m * (a.h >> 4) + unit, ss);
}

// One output element pair of a unit: row m, column c of the 16-column tile(s).  v0/v1 are the
// fp32 results of the unit's first/second tile.  The 16 lanes c = 0..15 of a row are adjacent
// lanes of one wave (RESID reduces over them).  Not for LM, whose callers keep a running arg-max.
template <int EPI, bool COH = false>
__device__ __forceinline__ void epilogue(const FusedGemmArgs &a, int unit, int m, int c, bool valid, float v0, float v1, float rs)
{
    if (EPI == FEPI_STORE) {
        if (valid) a.out[(size_t)m * a.Ntot + unit * 16 + c] = v0;
    } else if (EPI == FEPI_RESID) {
        const int n = unit * 16 + c;
        resid1<COH>(a, unit, m, c, valid, v0, valid ? ld<COH>(a.X + (size_t)m * a.h + n) : 0.f, valid ? a.gamma_next[n] : (uint16_t)0);
    } else if (EPI == FEPI_QKV) {
        if (!valid) return;
        const int TH = a.d >> 4, per_head = TH >> 1;
        int head = unit / per_head;
        const int pair = unit % per_head;
        v0 *= rs;
        v1 *= rs;
        const int b = a.by_k1(m), j = m - b * (a.k + 1);
        const int base = a.pos_base[b];                 // < 0: a rejected sequence, which must not touch the cache
        const int pos = base + j;                       // cache row of node j
        const int half = a.d >> 1, ch = pair * 16 + c;  // channel of v0; v1 is ch + half
        if (head < a.nq + a.nkv) {
            const float2 cs = *reinterpret_cast<const float2 *>(a.rope_cs + ((size_t)a.rope_pos[m] * half + ch) * 2);
            const float y0 = v0 * cs.x - v1 * cs.y, y1 = v0 * cs.y + v1 * cs.x;
            if (head < a.nq) {
                const int g = (int)a.by_g.d, kvh = a.by_g(head), hl = head - kvh * g, rr = j * g + hl;
                const size_t qs = ((size_t)b * a.nkv + kvh) * a.q_rows_pad * a.d;
                uint16_t h0, l0, h1, l1;
                split_bf16(y0, h0, l0);
                split_bf16(y1, h1, l1);
                const size_t i_0 = qs + packed_index(rr, ch, a.d >> 5), i_1 = qs + packed_index(rr, ch + half, a.d >> 5);
                st<COH>(a.Qp + i_0, h0); st<COH>(a.Qp_lo + i_0, l0);
                st<COH>(a.Qp + i_1, h1); st<COH>(a.Qp_lo + i_1, l1);
            } else if (base >= 0) {
                head -= a.nq;
                uint16_t *kk = a.Kc + kv_block_offset(a.kv, kv_page(a.kv, b, pos >> 5), head);
                st<COH>(kk + kblock_index(pos & 31, ch, a.d), f32_to_bf16(y0));
                st<COH>(kk + kblock_index(pos & 31, ch + half, a.d), f32_to_bf16(y1));
            }
        } else if (base >= 0) {
            head -= a.nq + a.nkv;
            uint16_t *vv = a.Vc + kv_block_offset(a.kv, kv_page(a.kv, b, pos >> 5), head);
            st<COH>(vv + vblock_index(pos & 31, ch, a.d), f32_to_bf16(v0));
            st<COH>(vv + vblock_index(pos & 31, ch + half, a.d), f32_to_bf16(v1));
        }
    } else if (EPI == FEPI_SWIGLU) {
        if (!valid) return;
        const float gt = v0 * rs, up = v1 * rs;
        const float hval = gt / (1.f + __expf(-gt)) * up;
        uint16_t hi, lo;
        split_bf16(hval, hi, lo);
        const size_t idx = packed_index(m, unit * 16 + c, a.KT_out);
        st<COH>(a.out_hi + idx, hi);
        st<COH>(a.out_lo + idx, lo);
    }
}

// Running arg-max of a row: the larger value, of equal ones the lower column.  A value that is no number never wins.
struct Best {
    float v;
    int i;
    __device__ __forceinline__ void take(float v2, int i2)
    {
        if (v2 > v || (v2 == v && i2 < i)) { v = v2; i = i2; }
    }
    static __device__ __forceinline__ Best none() { return Best{-INFINITY, 0x7FFFFFFF}; }
    __device__ __forceinline__ void across(int off) { take(__shfl_xor(v, off), __shfl_xor(i, off)); }   // the lane `off` away
};

// Sums over the 16 lanes of a row of lanes and over the whole wave, in every lane, without LDS.
__device__ __forceinline__ float row16_sum(float x)
{
    x += bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x128, 0xF, 0xF, true));   // rotated by 8, 4, 2, 1 lanes
    x += bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x124, 0xF, 0xF, true));
    x += bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x122, 0xF, 0xF, true));
    x += bits_f32((uint32_t)__builtin_amdgcn_mov_dpp((int)f32_bits(x), 0x121, 0xF, 0xF, true));
    return x;
}
__device__ __forceinline__ float wave_sum(float x)
{
    x = row16_sum(x);
    auto h = __builtin_amdgcn_permlane16_swap(f32_bits(x), f32_bits(x), false, false);
    x = bits_f32(h[0]) + bits_f32(h[1]);
    h = __builtin_amdgcn_permlane32_swap(f32_bits(x), f32_bits(x), false, false);
    return bits_f32(h[0]) + bits_f32(h[1]);
}

// rsqrt(mean(x^2) + eps) of row m from the producer's sums of squares; whole wave.  (The last workgroup of pgemm_kernel's split.)
template <bool COH = false> __device__ __forceinline__ float row_rstd(const FusedGemmArgs &a, int m, int lane)
{
    const int NSS = a.nss_in;
    float sum = 0.f;
    if (m < a.M)
        for (int t = lane; t < NSS; t += 64) sum += ld<COH>(a.ssq_in + (size_t)m * NSS + t);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    return rsqrtf(sum / (float)a.h + a.eps);
}

// ---- eight columns per thread ----
struct Vec8 {
    float v[8];
};

template <bool COH = false> __device__ __forceinline__ Vec8 load8(const float *p)
{
    if (COH) {   // device-scope: four 8-byte loads
        Vec8 r;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned long long u = ld<true>(reinterpret_cast<const unsigned long long *>(p) + q);
            r.v[2 * q] = __uint_as_float((uint32_t)u);
            r.v[2 * q + 1] = __uint_as_float((uint32_t)(u >> 32));
        }
        return r;
    }
    const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
    return Vec8{{a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]}};
}

template <bool COH = false> __device__ __forceinline__ void store8(float *p, const Vec8 &x)
{
    if (COH) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            st<true>(reinterpret_cast<unsigned long long *>(p) + q,
                     (unsigned long long)__float_as_uint(x.v[2 * q]) | ((unsigned long long)__float_as_uint(x.v[2 * q + 1]) << 32));
        return;
    }
    *reinterpret_cast<f32x4 *>(p) = f32x4{x.v[0], x.v[1], x.v[2], x.v[3]};
    *reinterpret_cast<f32x4 *>(p + 4) = f32x4{x.v[4], x.v[5], x.v[6], x.v[7]};
}

template <bool COH = false> __device__ __forceinline__ void st_record(uint16_t *p, const u32x4 &r)
{
    if (COH) {
        st<true>(reinterpret_cast<unsigned long long *>(p), (unsigned long long)r[0] | ((unsigned long long)r[1] << 32));
        st<true>(reinterpret_cast<unsigned long long *>(p) + 1, (unsigned long long)r[2] | ((unsigned long long)r[3] << 32));
        return;
    }
    *reinterpret_cast<u32x4 *>(p) = r;
}

// x[0..7] -> one lane record of bf16 hi parts and one of lo parts
__device__ __forceinline__ void split8(const Vec8 &x, u32x4 &hi, u32x4 &lo)
{
    uint32_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split_bf16x2(x.v[2 * e], x.v[2 * e + 1], h[e], l[e]);
    hi = u32x4{h[0], h[1], h[2], h[3]};
    lo = u32x4{l[0], l[1], l[2], l[3]};
}

__device__ __forceinline__ u32x4 round8(const Vec8 &x)
{
    return u32x4{pack_bf16x2(x.v[0], x.v[1]), pack_bf16x2(x.v[2], x.v[3]), pack_bf16x2(x.v[4], x.v[5]), pack_bf16x2(x.v[6], x.v[7])};
}

// Sums of the J slices of 8 columns each at `col` (and at `col1`, with TWO) of row m, slices in order.  BATCH slices are
// fetched at a time: one by one, every slice is a memory round trip of its own.
template <int BATCH, bool TWO, bool COH = false>
__device__ __forceinline__ void sum_slices(const FusedGemmArgs &a, int m, int col, int col1, Vec8 &s0, Vec8 &s1)
{
    const float *p = a.partials + (size_t)m * a.Ntot + col, *p1 = a.partials + (size_t)m * a.Ntot + col1;
    const size_t jstride = (size_t)a.part_rows * a.Ntot;
    for (int j0 = 0; j0 < a.J; j0 += BATCH) {
        Vec8 t0[BATCH], t1[BATCH];
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
            if (j0 + u < a.J) {
                t0[u] = load8<COH>(p + (j0 + u) * jstride);
                if (TWO) t1[u] = load8<COH>(p1 + (j0 + u) * jstride);
            }
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
            if (j0 + u < a.J) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    s0.v[e] = j0 + u ? s0.v[e] + t0[u].v[e] : t0[u].v[e];
                    if (TWO) s1.v[e] = j0 + u ? s1.v[e] + t1[u].v[e] : t1[u].v[e];
                }
            }
    }
}

// Epilogues on 8 consecutive columns per thread, which are one 16-byte lane record of a packed operand.

// RESID: X += v0, packed X * gamma.  v0 = the projection's result at columns col..col+7 of row m.  Returns the sum of squares
// of the updated columns.
template <bool COH> __device__ __forceinline__ float resid8(const FusedGemmArgs &a, int m, int col, const Vec8 &v0)
{
    const Vec8 x = load8<COH>(a.X + (size_t)m * a.h + col);
    u32x4 gamma;
    __builtin_memcpy(&gamma, a.gamma_next + col, 16);   // caller's array: no alignment assumed
    float ss = 0.f;
    Vec8 xn, xg;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        xn.v[e] = x.v[e] + v0.v[e];
        xg.v[e] = xn.v[e] * bits_f32(e & 1 ? gamma[e >> 1] & 0xFFFF0000u : gamma[e >> 1] << 16);
        ss += xn.v[e] * xn.v[e];
    }
    store8<COH>(a.X + (size_t)m * a.h + col, xn);
    u32x4 hi, lo;
    split8(xg, hi, lo);
    const size_t idx = packed_index(m, col, (a.h + 31) >> 5);
    st_record<COH>(a.out_hi + idx, hi);
    st_record<COH>(a.out_lo + idx, lo);
    return ss;
}

// RESID with one sum of squares per 16 columns; whole waves call it.  kg: which 8-column group of its 32-column block the
// thread holds (lanes kg and kg^1, 16 lanes apart, share a sum).
template <bool COH> __device__ __forceinline__ void resid_block(const FusedGemmArgs &a, int m, int col, bool live, int kg, const Vec8 &v0)
{
    float ss = live ? resid8<COH>(a, m, col, v0) : 0.f;
    ss += __shfl_xor(ss, 16);   // the other 8 columns of the 16-column group
    if (live && !(kg & 1)) st<COH>(a.ssq_out + (size_t)m * (a.h >> 4) + (col >> 4), ss);
}

// QKV: v0 at channels ch..ch+7 of the first half of a head, v1 at the same channels of the second half.
__device__ __forceinline__ void qkv8(const FusedGemmArgs &a, int m, int head, int ch, float rs, Vec8 v0, Vec8 v1)
{
    const int half = a.d >> 1;
    const int b = a.by_k1(m), j = m - b * (a.k + 1);
    const int base = a.pos_base[b];               // cache row of the sequence's first node; < 0: a rejected sequence, which must not touch the cache
    const int pos = base + j;                     // cache row of node j
#pragma unroll
    for (int e = 0; e < 8; ++e) { v0.v[e] *= rs; v1.v[e] *= rs; }
    if (head < a.nq + a.nkv) {
        const float *cs = a.rope_cs + ((size_t)a.rope_pos[m] * half + ch) * 2;
        const Vec8 cs0 = load8(cs), cs1 = load8(cs + 8);   // (cos, sin) of channels ch..ch+3, ch+4..ch+7
        Vec8 y0, y1;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float co = e < 4 ? cs0.v[2 * e] : cs1.v[2 * (e - 4)], si = e < 4 ? cs0.v[2 * e + 1] : cs1.v[2 * (e - 4) + 1];
            y0.v[e] = v0.v[e] * co - v1.v[e] * si;
            y1.v[e] = v0.v[e] * si + v1.v[e] * co;
        }
        if (head < a.nq) {
            const int g = (int)a.by_g.d, kvh = a.by_g(head), hl = head - kvh * g, rr = j * g + hl;
            const size_t qs = ((size_t)b * a.nkv + kvh) * a.q_rows_pad * a.d;
            u32x4 h0, l0, h1, l1;
            split8(y0, h0, l0);
            split8(y1, h1, l1);
            const size_t i_0 = qs + packed_index(rr, ch, a.d >> 5), i_1 = qs + packed_index(rr, ch + half, a.d >> 5);
            *reinterpret_cast<u32x4 *>(a.Qp + i_0) = h0; *reinterpret_cast<u32x4 *>(a.Qp_lo + i_0) = l0;
            *reinterpret_cast<u32x4 *>(a.Qp + i_1) = h1; *reinterpret_cast<u32x4 *>(a.Qp_lo + i_1) = l1;
        } else if (base >= 0) {
            head -= a.nq;
            uint16_t *kk = a.Kc + kv_block_offset(a.kv, kv_page(a.kv, b, pos >> 5), head);
            *reinterpret_cast<u32x4 *>(kk + kblock_index(pos & 31, ch, a.d)) = round8(y0);
            *reinterpret_cast<u32x4 *>(kk + kblock_index(pos & 31, ch + half, a.d)) = round8(y1);
        }
    } else if (base >= 0) {
        head -= a.nq + a.nkv;
        uint16_t *vv = a.Vc + kv_block_offset(a.kv, kv_page(a.kv, b, pos >> 5), head);
        const u32x4 r0 = round8(v0), r1 = round8(v1);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            vv[vblock_index(pos & 31, ch + e, a.d)] = (uint16_t)(r0[e >> 1] >> (e & 1) * 16);
            vv[vblock_index(pos & 31, ch + half + e, a.d)] = (uint16_t)(r1[e >> 1] >> (e & 1) * 16);
        }
    }
}

// SWIGLU: gate v0, up v1 at columns col..col+7 of the FFN.
__device__ __forceinline__ void swiglu8(const FusedGemmArgs &a, int m, int col, float rs, const Vec8 &v0, const Vec8 &v1)
{
    Vec8 hv;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float gg = v0.v[e] * rs;
        hv.v[e] = gg / (1.f + __expf(-gg)) * (v1.v[e] * rs);
    }
    u32x4 hi, lo;
    split8(hv, hi, lo);
    const size_t idx = packed_index(m, col, a.KT_out);
    *reinterpret_cast<u32x4 *>(a.out_hi + idx) = hi;
    *reinterpret_cast<u32x4 *>(a.out_lo + idx) = lo;
}

// LM: logits (if asked for), and columns n0..n0+7 of row m into the row's running arg-max.
__device__ __forceinline__ void lm8(const FusedGemmArgs &a, int m, int n0, float rs, Vec8 v0, Best &best)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v0.v[e] *= rs;
        best.take(v0.v[e], n0 + e);
    }
    if (a.logits) store8(a.logits + (size_t)m * a.vocab + n0, v0);
}

// ---- four columns per lane ----
// qgemm16_kernel multiplies weights x activations, so a lane holds columns 4*(l/16)..+3 of row l%16 of every 16 x 16 tile: the
// epilogues below work on the accumulators as they are.  What they read from memory can be requested ahead.  Args: the fields of
// FusedGemmArgs that they read.
struct QuadIn {
    f32x4 x0, x1;       // RESID: residual of both tiles; QKV: (cos, sin) of channels 0, 1 and of 2, 3
    uint2 g0, g1;       // RESID: gains of both tiles
    int base;           // QKV: cache row of the sequence's first node; < 0: a rejected sequence, which must not touch the cache
};

__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
__device__ __forceinline__ void split4(const f32x4 &x, uint2 &hi, uint2 &lo)
{
    split_bf16x2(x[0], x[1], hi.x, lo.x);
    split_bf16x2(x[2], x[3], hi.y, lo.y);
}
__device__ __forceinline__ uint2 round4(const f32x4 &x) { return uint2{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])}; }

// Lanes kg and kg + 1 (16 apart, kg even) hold columns 0..3 and 4..7 of one 16-byte record: returns, to the first, the record of x,
// to the second that of y, and stores them at p and q.  Stored by halves, every line would be written twice.
__device__ __forceinline__ void store_records(uint16_t *p, uint16_t *q, const uint2 &x, const uint2 &y, bool first)
{
    const auto a = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false), b = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    *reinterpret_cast<u32x4 *>(first ? p : q) = u32x4{a[0], b[0], a[1], b[1]};
}

// Sum over the four lanes 16 apart that share a row, in each of them.
__device__ __forceinline__ float row_sum4(float x)
{
    auto h = __builtin_amdgcn_permlane16_swap(f32_bits(x), f32_bits(x), false, false);
    x = bits_f32(h[0]) + bits_f32(h[1]);
    h = __builtin_amdgcn_permlane32_swap(f32_bits(x), f32_bits(x), false, false);
    return bits_f32(h[0]) + bits_f32(h[1]);
}

// RESID: X += v, packed X * gamma at columns col..col+3 of row m.  Returns the sum of squares of the updated columns.
// (m, col / 8) are the same in the two lanes of a pair, and both call it: so with all below.
template <typename Args> __device__ __forceinline__ float resid4(const Args &a, int m, int col, const f32x4 &v, const f32x4 &x, const uint2 &gamma)
{
    const f32x4 xn = x + v;
    const f32x4 g = {bits_f32(gamma.x << 16), bits_f32(gamma.x & 0xFFFF0000u), bits_f32(gamma.y << 16), bits_f32(gamma.y & 0xFFFF0000u)};
    *reinterpret_cast<f32x4 *>(a.X + (size_t)m * a.h + col) = xn;
    uint2 hi, lo;
    split4(xn * g, hi, lo);
    const size_t idx = packed_index(m, col & ~7, (a.h + 31) >> 5);
    store_records(a.out_hi + idx, a.out_lo + idx, hi, lo, !(col & 4));
    return (xn[0] * xn[0] + xn[1] * xn[1]) + (xn[2] * xn[2] + xn[3] * xn[3]);
}

// QKV: v0 at channels ch..ch+3 of the first half of a head, v1 at the same channels of the second half.
template <typename Args> __device__ __forceinline__ void qkv4(const Args &a, int m, int head, int ch, float rs, f32x4 v0, f32x4 v1, const QuadIn &in)
{
    const int half = a.d >> 1;
    const int b = a.by_k1(m), j = m - b * (a.k + 1);
    const int pos = in.base + j;                  // cache row of node j
    v0 *= rs;
    v1 *= rs;
    if (head < a.nq + a.nkv) {
        const f32x4 co = {in.x0[0], in.x0[2], in.x1[0], in.x1[2]}, si = {in.x0[1], in.x0[3], in.x1[1], in.x1[3]};
        const f32x4 y0 = v0 * co - v1 * si, y1 = v0 * si + v1 * co;
        if (head < a.nq) {
            const int g = (int)a.by_g.d, kvh = a.by_g(head), hl = head - kvh * g, rr = j * g + hl;
            const size_t qs = ((size_t)b * a.nkv + kvh) * a.q_rows_pad * a.d;
            uint2 h0, l0, h1, l1;
            split4(y0, h0, l0);
            split4(y1, h1, l1);
            const size_t i_0 = qs + packed_index(rr, ch & ~7, a.d >> 5), i_1 = qs + packed_index(rr, (ch & ~7) + half, a.d >> 5);
            store_records(a.Qp + i_0, a.Qp_lo + i_0, h0, l0, !(ch & 4));
            store_records(a.Qp + i_1, a.Qp_lo + i_1, h1, l1, !(ch & 4));
        } else if (in.base >= 0) {
            head -= a.nq;
            uint16_t *kk = a.Kc + kv_block_offset(a.kv, kv_page(a.kv, b, pos >> 5), head);
            store_records(kk + kblock_index(pos & 31, ch & ~7, a.d), kk + kblock_index(pos & 31, (ch & ~7) + half, a.d), round4(y0), round4(y1), !(ch & 4));
        }
    } else if (in.base >= 0) {
        head -= a.nq + a.nkv;
        uint16_t *vv = a.Vc + kv_block_offset(a.kv, kv_page(a.kv, b, pos >> 5), head);
        const uint2 r0 = round4(v0), r1 = round4(v1);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            vv[vblock_index(pos & 31, ch + e, a.d)] = (uint16_t)((e < 2 ? r0.x : r0.y) >> (e & 1) * 16);
            vv[vblock_index(pos & 31, ch + half + e, a.d)] = (uint16_t)((e < 2 ? r1.x : r1.y) >> (e & 1) * 16);
        }
    }
}

// SWIGLU: gate v0, up v1 at columns col..col+3 of the FFN.
template <typename Args> __device__ __forceinline__ void swiglu4(const Args &a, int m, int col, float rs, const f32x4 &v0, const f32x4 &v1)
{
    f32x4 hv;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float gg = v0[e] * rs;
        hv[e] = gg / (1.f + __expf(-gg)) * (v1[e] * rs);
    }
    uint2 hi, lo;
    split4(hv, hi, lo);
    const size_t idx = packed_index(m, col & ~7, a.KT_out);
    store_records(a.out_hi + idx, a.out_lo + idx, hi, lo, !(col & 4));
}

// LM: logits (if asked for), and columns n0..n0+3 of row m into the row's running arg-max.
template <typename Args> __device__ __forceinline__ void lm4(const Args &a, int m, int n0, float rs, f32x4 v, Best &best)
{
    v *= rs;
#pragma unroll
    for (int e = 0; e < 4; ++e) best.take(v[e], n0 + e);
    if (a.logits) *reinterpret_cast<f32x4 *>(a.logits + (size_t)m * a.vocab + n0) = v;
}

}  // namespace
