// attention.hip -- multi-head scaled dot-product attention, forward and
// backward, for fp32 partitions (head width <= 64, a multiple of 4; lengths up
// to 1024).
//
// A = softmax(Q K^T s + mask), O = A V per (sequence, head), s = 1/sqrt(d_h);
// the causal mask removes keys j > i.  A workgroup of four waves owns 16 rows
// of one (sequence, head): query rows (forward, dQ) or key rows (dK, dV).  The
// backward is split into a query-row pass (dQ, and delta_i = rowsum(dO_i O_i))
// and a key-row pass (dK, dV) so that no two workgroups add into the same
// output: results are deterministic and the re-materialised forward
// reproduces the first pass.
//
// The products run on v_mfma_f32_16x16x4_f32, which adds its four products one
// after the other, each rounded: an fma chain in k order.  Phase one: the waves
// share out the 16 x 16 blocks of scores (chains over the head width) and leave
// them in LDS; between: the row softmax, one wave per row, lane l over columns
// l, l + 64, ..; phase two: each wave runs one 16-column block of the output, a
// chain over all columns of the score rows.  What bounds a workgroup is phase
// two's chain (about 70 cycles per four columns), which is why the rows per
// workgroup are few.  Each result equals, bit for bit, that of the form this
// replaced -- a wave per row with scalar fma chains, every lane reading whole
// K and V rows from memory: at 4 x 8 heads of 128 x 64, in a step, forward 45.5
// -> 13.7 us, dQ 55.9 -> 20.7, dK/dV 77.2 -> 19.5.  That includes infinities and
// NaN behind the causal mask: a product's 16 x 16 block on the diagonal multiplies
// them by the masked scores' zeros, so where such a block holds any, its chain
// leaves the masked products out one by one (masked_block).
//
// bf16 partitions use the MFMA kernels in attention_mfma.hip.
#include "common.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"

namespace gp {

namespace {

constexpr int RB = 16;      // rows per workgroup
constexpr int MAXS = 1024;  // longest key / query row held in LDS

__device__ __forceinline__ f32x4 mma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// 4 x 4 transpose of v[e] over the four 16-lane groups: element e of group s
// becomes element s of group e.
__device__ __forceinline__ void transpose4(float* v) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto swap32 = [](float& a, float& b) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    auto swap16 = [](float& a, float& b) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        a = __uint_as_float(r[0]);
        b = __uint_as_float(r[1]);
    };
    swap32(v[0], v[2]);
    swap32(v[1], v[3]);
    swap16(v[0], v[1]);
    swap16(v[2], v[3]);
#endif
}

// MFMA operand of one row (lane % 16 of a 16-row block; `row` its address) over
// the head width: f[4 t + e] is feature 16 t + 4 e + lane / 16, zero beyond dh.
template <int TD>
__device__ __forceinline__ void row_frag(const float* row, int dh, int lane, float* f) {
#pragma unroll
    for (int t = 0; t < TD; ++t) {
        const int d = 16 * t + 4 * (lane >> 4);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (d < dh) v = *reinterpret_cast<const f32x4*>(row + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) f[4 * t + e] = v[e];
        transpose4(f + 4 * t);
    }
}
template <int TD>
__device__ __forceinline__ f32x4 block_dot(const float* a, const float* b) {
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4 * TD; ++i) c = mma4(a[i], b[i], c);
    return c;
}

// Row stride of the score rows in LDS: 16 rows x 4 consecutive columns then
// fall in distinct banks.
constexpr int srow(int SB) { return SB + 4; }

// This lane's column of the rows of X: element k is row k's, zero from row n on
// (out of the buffer's range).
struct XCol {
    Rsrc r;
    uint32_t off, ld;  // bytes
    __device__ __forceinline__ float operator[](int k) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off + k * ld, 0, 0));
    }
};
__device__ __forceinline__ XCol x_col(const float* X, long ld, int n, int dh, int col) {
    return {make_rsrc(X, (uint32_t)(((long)(n - 1) * ld + dh) * 4)), (uint32_t)min(col, dh - 1) * 4, (uint32_t)ld * 4};
}

// sum over k in [k0, k1) of P[16][k] X[k][col] (k0 a multiple of 4): lane's
// score row lane % 16, this lane's column of X, whose rows end at k1.  P is zero
// from k1 to the next multiple of 4.  X does not depend on the scores: the first
// 4 NPRE rows are loaded before they are ready (prefetch_rows).
constexpr int NPRE = 32;
__device__ __forceinline__ void prefetch_rows(const XCol& x, int k0, int k1, int lane, float* pre) {
#pragma unroll
    for (int i = 0; i < NPRE; ++i) {
        pre[i] = 0.f;
        if (k0 + 4 * i < k1) pre[i] = x[k0 + 4 * i + (lane >> 4)];
    }
}
template <int SB>
__device__ __forceinline__ f32x4 chain(const float* P, const XCol& x, int k0, int k1, int lane, const float* pre) {
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    const float* p = P + (lane & 15) * srow(SB) + (lane >> 4);
#pragma unroll
    for (int i = 0; i < NPRE; ++i)
        if (k0 + 4 * i < k1) c = mma4(p[k0 + 4 * i], pre[i], c);
#pragma unroll 16
    for (int k = k0 + 4 * NPRE; k < k1; k += 4) c = mma4(p[k], x[k + (lane >> 4)], c);
    return c;
}
// Whether any X row of the diagonal block [d, d + 16) holds an infinity or a NaN
// in the wave's columns (the same answer in every lane).
__device__ __forceinline__ bool masked_block(const XCol& x, int d, int lane) {
    bool bad = false;
#pragma unroll
    for (int t = 0; t < 4; ++t) bad = bad || !(fabsf(x[d + 4 * t + (lane >> 4)]) < INFINITY);
    return __any(bad);
}
// The same sum where masked_block holds: of the block's columns, row r of the 16
// takes only d .. d + r (UPTO) or d + r .. d + 15, as scalar fma chains in the same
// order.
template <int SB, bool UPTO>
__device__ __forceinline__ f32x4 chain_masked(const float* P, const XCol& x, int k0, int k1, int d, int lane) {
    f32x4 c = {0.f, 0.f, 0.f, 0.f};
    const float* p = P + (lane & 15) * srow(SB) + (lane >> 4);
#pragma unroll 1
    for (int k = k0; k < d; k += 4) c = mma4(p[k], x[k + (lane >> 4)], c);
#pragma unroll 1
    for (int k = d; k < min(d + 16, k1); ++k) {
        const float v = x[k];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * (lane >> 4) + r;
            if (UPTO ? k - d <= row : k - d >= row) c[r] = __builtin_fmaf(P[row * srow(SB) + k], v, c[r]);
        }
    }
#pragma unroll 1
    for (int k = d + 16; k < k1; k += 4) c = mma4(p[k], x[k + (lane >> 4)], c);
    return c;
}

// Workgroup -> row block and (sequence, head).
struct Place {
    int r0, h, b;
    long bh;
};
__device__ __forceinline__ Place place(const AttnArgs& a, int rows) {
    const int nb = (rows + RB - 1) / RB;
    Place p;
    p.bh = blockIdx.x / nb;
    p.r0 = (int)(blockIdx.x % nb) * RB;
    p.h = (int)(p.bh % a.H);
    p.b = (int)(p.bh / a.H);
    return p;
}

template <int SB, int TD>
__global__ void __launch_bounds__(256) attn_fwd_f32(AttnArgs a) {
    __shared__ float ps[RB * srow(SB)];
    __shared__ float sums[RB];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const Place pl = place(a, a.Sq);
    const float* Q = reinterpret_cast<const float*>(a.q) + (long)pl.b * a.Sq * a.ldq + pl.h * a.dh;
    const float* K = reinterpret_cast<const float*>(a.k) + (long)pl.b * a.Sk * a.ldk + pl.h * a.dh;
    const float* V = reinterpret_cast<const float*>(a.v) + (long)pl.b * a.Sk * a.ldv + pl.h * a.dh;
    const int len = a.causal ? min(a.Sk, pl.r0 + RB) : a.Sk;  // columns any row of the block uses
    float qf[4 * TD];
    row_frag<TD>(Q + (long)min(pl.r0 + (lane & 15), a.Sq - 1) * a.ldq, a.dh, lane, qf);
    for (int kb = w * 16; kb < len; kb += 64) {
        float kf[4 * TD];
        row_frag<TD>(K + (long)min(kb + (lane & 15), a.Sk - 1) * a.ldk, a.dh, lane, kf);
        const f32x4 c = block_dot<TD>(qf, kf);
#pragma unroll
        for (int r = 0; r < 4; ++r) ps[(4 * (lane >> 4) + r) * srow(SB) + kb + (lane & 15)] = a.scale * c[r];
    }
    const int col = w * 16 + (lane & 15);
    const XCol x = x_col(V, a.ldv, len, a.dh, col);
    float pre[NPRE];
    prefetch_rows(x, 0, len, lane, pre);
    __syncthreads();
    {
        // the wave's four rows side by side, so that their reductions overlap
        float* p = ps + w * 4 * srow(SB);
        int jm[4];
        float m[4], sum[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            jm[r] = a.causal ? min(pl.r0 + w * 4 + r + 1, a.Sk) : a.Sk;
            m[r] = -INFINITY;
            sum[r] = 0.f;
        }
        for (int j = lane; j < len; j += 64)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (j < jm[r]) m[r] = fmaxf(m[r], p[r * srow(SB) + j]);
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = wave_max(m[r]);
        for (int j = lane; j < ((len + 3) & ~3); j += 64)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float e = 0.f;
                if (j < jm[r]) {
                    e = expf(p[r * srow(SB) + j] - m[r]);
                    sum[r] += e;
                }
                p[r * srow(SB) + j] = e;
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] = wave_sum(sum[r]);
        if (lane == 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = pl.r0 + w * 4 + r;
                sums[w * 4 + r] = sum[r];
                if (a.lse && i < a.Sq) a.lse[pl.bh * a.Sq + i] = m[r] + logf(sum[r]);
            }
    }
    __syncthreads();
    if (w * 16 >= a.dh) return;
    const f32x4 o = a.causal && masked_block(x, pl.r0, lane) ? chain_masked<SB, true>(ps, x, 0, len, pl.r0, lane)
                                                             : chain<SB>(ps, x, 0, len, lane, pre);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int rr = 4 * (lane >> 4) + r, i = pl.r0 + rr;
        if (i < a.Sq && col < a.dh)
            reinterpret_cast<float*>(a.o)[((long)pl.b * a.Sq + i) * a.ldo + pl.h * a.dh + col] = o[r] / sums[rr];
    }
}

// dQ pass: 16 query rows.
template <int SB, int TD>
__global__ void __launch_bounds__(256) attn_bwd_dq_f32(AttnArgs a) {
    __shared__ float ds[RB * srow(SB)];
    __shared__ float dl[RB], ls[RB];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const Place pl = place(a, a.Sq);
    const long q0 = (long)pl.b * a.Sq;
    const int ho = pl.h * a.dh;
    const float* K = reinterpret_cast<const float*>(a.k) + (long)pl.b * a.Sk * a.ldk + ho;
    const float* V = reinterpret_cast<const float*>(a.v) + (long)pl.b * a.Sk * a.ldv + ho;
    const int len = a.causal ? min(a.Sk, pl.r0 + RB) : a.Sk;
    float od[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = pl.r0 + w * 4 + r;
        od[r] = 0.f;
        if (lane < a.dh && i < a.Sq)
            od[r] = reinterpret_cast<const float*>(a.dout)[(q0 + i) * a.lddo + ho + lane] *
                    reinterpret_cast<const float*>(a.o)[(q0 + i) * a.ldo + ho + lane];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) od[r] = wave_sum(od[r]);
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = pl.r0 + w * 4 + r;
            if (i >= a.Sq) break;
            dl[w * 4 + r] = od[r];
            ls[w * 4 + r] = a.lse[pl.bh * a.Sq + i];
            a.delta[pl.bh * a.Sq + i] = od[r];
        }
    const long qrow = q0 + min(pl.r0 + (lane & 15), a.Sq - 1);
    float qf[4 * TD], gf[4 * TD];
    row_frag<TD>(reinterpret_cast<const float*>(a.q) + qrow * a.ldq + ho, a.dh, lane, qf);
    row_frag<TD>(reinterpret_cast<const float*>(a.dout) + qrow * a.lddo + ho, a.dh, lane, gf);
    __syncthreads();
    for (int kb = w * 16; kb < ((len + 3) & ~3); kb += 64) {
        const long krow = min(kb + (lane & 15), a.Sk - 1);
        float kf[4 * TD], vf[4 * TD];
        row_frag<TD>(K + krow * a.ldk, a.dh, lane, kf);
        row_frag<TD>(V + krow * a.ldv, a.dh, lane, vf);
        const f32x4 c = block_dot<TD>(qf, kf), g = block_dot<TD>(gf, vf);
        const int j = kb + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = 4 * (lane >> 4) + r, i = pl.r0 + rr;
            float x = 0.f;
            if (i < a.Sq && j < (a.causal ? min(i + 1, a.Sk) : a.Sk)) {
                const float p = expf(a.scale * c[r] - ls[rr]);
                x = p * (g[r] - dl[rr]);
            }
            ds[rr * srow(SB) + j] = x;
        }
    }
    const int col = w * 16 + (lane & 15);
    const XCol x = x_col(K, a.ldk, len, a.dh, col);
    float pre[NPRE];
    prefetch_rows(x, 0, len, lane, pre);
    __syncthreads();
    if (w * 16 >= a.dh) return;
    const f32x4 g = a.causal && masked_block(x, pl.r0, lane) ? chain_masked<SB, true>(ds, x, 0, len, pl.r0, lane)
                                                             : chain<SB>(ds, x, 0, len, lane, pre);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int i = pl.r0 + 4 * (lane >> 4) + r;
        if (i < a.Sq && col < a.dh) reinterpret_cast<float*>(a.dq)[(q0 + i) * a.lddq + ho + col] = a.scale * g[r];
    }
}

// dK, dV pass: 16 key rows.
template <int SB, int TD>
__global__ void __launch_bounds__(256) attn_bwd_dkv_f32(AttnArgs a) {
    __shared__ float ps[RB * srow(SB)], ds[RB * srow(SB)];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const Place pl = place(a, a.Sk);
    const long k0 = (long)pl.b * a.Sk;
    const int ho = pl.h * a.dh;
    const float* Q = reinterpret_cast<const float*>(a.q) + (long)pl.b * a.Sq * a.ldq + ho;
    const float* G = reinterpret_cast<const float*>(a.dout) + (long)pl.b * a.Sq * a.lddo + ho;
    const float* lse = a.lse + pl.bh * a.Sq;
    const float* delta = a.delta + pl.bh * a.Sq;
    const int first = a.causal ? pl.r0 : 0;  // queries before it see none of these keys (r0 % 16 == 0)
    const long krow = k0 + min(pl.r0 + (lane & 15), a.Sk - 1);
    float kf[4 * TD], vf[4 * TD];
    row_frag<TD>(reinterpret_cast<const float*>(a.k) + krow * a.ldk + ho, a.dh, lane, kf);
    row_frag<TD>(reinterpret_cast<const float*>(a.v) + krow * a.ldv + ho, a.dh, lane, vf);
    for (int qb = first + w * 16; qb < ((a.Sq + 3) & ~3); qb += 64) {
        const int i = qb + (lane & 15);
        const long qrow = min(i, a.Sq - 1);
        float qf[4 * TD], gf[4 * TD];
        row_frag<TD>(Q + qrow * a.ldq, a.dh, lane, qf);
        row_frag<TD>(G + qrow * a.lddo, a.dh, lane, gf);
        const float li = lse[qrow], di = delta[qrow];
        const f32x4 c = block_dot<TD>(kf, qf), g = block_dot<TD>(vf, gf);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int rr = 4 * (lane >> 4) + r, j = pl.r0 + rr;
            float p = 0.f, x = 0.f;
            if (i < a.Sq && (!a.causal || i >= j)) {
                p = expf(a.scale * c[r] - li);
                x = p * (g[r] - di);
            }
            ps[rr * srow(SB) + i] = p;
            ds[rr * srow(SB) + i] = x;
        }
    }
    const int col = w * 16 + (lane & 15);
    const XCol xg = x_col(G, a.lddo, a.Sq, a.dh, col), xq = x_col(Q, a.ldq, a.Sq, a.dh, col);
    float pre[NPRE], qpre[NPRE];
    prefetch_rows(xg, first, a.Sq, lane, pre);
    prefetch_rows(xq, first, a.Sq, lane, qpre);
    __syncthreads();
    if (w * 16 >= a.dh) return;
    const f32x4 gv = a.causal && masked_block(xg, first, lane) ? chain_masked<SB, false>(ps, xg, first, a.Sq, first, lane)
                                                               : chain<SB>(ps, xg, first, a.Sq, lane, pre);
    const f32x4 gk = a.causal && masked_block(xq, first, lane) ? chain_masked<SB, false>(ds, xq, first, a.Sq, first, lane)
                                                               : chain<SB>(ds, xq, first, a.Sq, lane, qpre);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int j = pl.r0 + 4 * (lane >> 4) + r;
        if (j < a.Sk && col < a.dh) {
            reinterpret_cast<float*>(a.dv)[(k0 + j) * a.lddv + ho + col] = gv[r];
            reinterpret_cast<float*>(a.dk)[(k0 + j) * a.lddk + ho + col] = a.scale * gk[r];
        }
    }
}

// KERNEL<SB, TD> for score rows of `len` columns and the head width.
#define GP_TD_SWITCH(SB, KERNEL, GRID)                                               \
    switch ((a.dh + 15) / 16) {                                                      \
    case 1: klaunch(KERNEL<SB, 1>, GRID, 256, 0, st, a); break;                      \
    case 2: klaunch(KERNEL<SB, 2>, GRID, 256, 0, st, a); break;                      \
    case 3: klaunch(KERNEL<SB, 3>, GRID, 256, 0, st, a); break;                      \
    default: klaunch(KERNEL<SB, 4>, GRID, 256, 0, st, a); break;                     \
    }
#define GP_SB_SWITCH(LEN, KERNEL, GRID)                                              \
    do {                                                                             \
        if ((LEN) <= 128) { GP_TD_SWITCH(128, KERNEL, GRID) }                        \
        else if ((LEN) <= 320) { GP_TD_SWITCH(320, KERNEL, GRID) }                   \
        else { GP_TD_SWITCH(1024, KERNEL, GRID) }                                    \
        GP_LAUNCH_CHECK();                                                           \
    } while (0)

bool f32_ok(const AttnArgs& a) { return a.dh <= 64 && a.dh % 4 == 0 && a.Sk <= MAXS && a.Sq <= MAXS; }

} // namespace

gp_status attention_fwd_f32(const AttnArgs& a, hipStream_t st) {
    if (!f32_ok(a)) return set_error(GP_ERR_UNSUPPORTED, "attention: d_h <= 64, a multiple of 4, and S <= 1024");
    GP_SB_SWITCH(a.Sk, attn_fwd_f32, (unsigned)((long)a.n * a.H * ((a.Sq + RB - 1) / RB)));
    return GP_OK;
}

gp_status attention_bwd_f32(const AttnArgs& a, hipStream_t st) {
    if (!f32_ok(a)) return set_error(GP_ERR_UNSUPPORTED, "attention: d_h <= 64, a multiple of 4, and S <= 1024");
    GP_SB_SWITCH(a.Sk, attn_bwd_dq_f32, (unsigned)((long)a.n * a.H * ((a.Sq + RB - 1) / RB)));
    GP_SB_SWITCH(a.Sq, attn_bwd_dkv_f32, (unsigned)((long)a.n * a.H * ((a.Sk + RB - 1) / RB)));
    return GP_OK;
}

} // namespace gp
