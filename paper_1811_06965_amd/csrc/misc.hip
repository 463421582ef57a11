#include <algorithm>
// misc.hip -- boundary intake, casts, loss heads and the synchronous update.
//
// All reductions are two-stage with a fixed order (per-block partials, then
// one finalising block), so every result is reproducible bit for bit.
#include "common.hpp"
#include "kernels.hpp"

namespace gp {

namespace {

constexpr int EW_BLOCKS = 1024;   // grid of the grid-stride elementwise kernels
constexpr int LOSS_BLOCKS = 256;  // partials of the MSE loss

template <typename T>
__global__ void __launch_bounds__(256) intake_kernel(const T* __restrict__ src, T* __restrict__ stash,
                                                     float* __restrict__ x32, long count) {
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long)gridDim.x * 256) {
        const T v = src[i];
        if (stash) stash[i] = v;
        if (x32) x32[i] = to_f32(v);
    }
}

// 8 bf16 elements per thread with 16-byte accesses (count % 8 == 0, aligned pointers).
__global__ void __launch_bounds__(256) intake_bf16_v8(const bf16x8* __restrict__ src, bf16x8* __restrict__ stash,
                                                      f32x4* __restrict__ x32, long n8) {
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n8; i += (long)gridDim.x * 256) {
        const bf16x8 v = src[i];
        if (stash) stash[i] = v;
        if (x32) {
            x32[2 * i] = f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
            x32[2 * i + 1] = f32x4{(float)v[4], (float)v[5], (float)v[6], (float)v[7]};
        }
    }
}

template <typename T>
__global__ void __launch_bounds__(256) cast_kernel(const float* __restrict__ src, T* __restrict__ dst, long count) {
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long)gridDim.x * 256)
        dst[i] = to_elt<T>(src[i]);
}

// Four elements per thread and access (count % 4 == 0; y, d32 and de are the
// library's aligned buffers, the caller's t may have any element alignment:
// tvec = 0 then).  At 512 rows of 512 the element-wise form took 13 us.
template <typename T>
__global__ void __launch_bounds__(256) mse_kernel(const float* __restrict__ y, const T* __restrict__ t, long count,
                                                  double norm, float* __restrict__ d32, T* __restrict__ de,
                                                  double* __restrict__ partial, int tvec) {
    typedef T T4 __attribute__((ext_vector_type(4)));
    __shared__ double red[4];
    double s = 0.0;
    const float scale = (float)(2.0 / norm);
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count / 4; i += (long)gridDim.x * 256) {
        const f32x4 yv = reinterpret_cast<const f32x4*>(y)[i];
        T4 tv;
        if (tvec)
            tv = reinterpret_cast<const T4*>(t)[i];
        else
            tv = T4{t[4 * i], t[4 * i + 1], t[4 * i + 2], t[4 * i + 3]};
        f32x4 g;
        T4 ge;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float d = yv[e] - to_f32(tv[e]);
            s += (double)d * (double)d;
            g[e] = scale * d;
            ge[e] = to_elt<T>(g[e]);
        }
        reinterpret_cast<f32x4*>(d32)[i] = g;
        reinterpret_cast<T4*>(de)[i] = ge;
    }
    s = wave_sum_d(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = (red[0] + red[1] + red[2] + red[3]) / norm;
}

// The mini-batch loss: `used` partials of each of M micro-batches (rows of
// `stride` doubles).  One block; thread t adds partials t, t + 1024, .. of the
// M used-long rows laid end to end, then the 1024 sums pair up in a fixed
// tree.  (One thread adding every micro-batch's partials after each backward
// took 16 us at 256 partials and 63 us at 1024, M times per step on the
// backward's own stream; this runs once, when the caller asks for the loss.)
__global__ void __launch_bounds__(1024) loss_finalize_kernel(const double* __restrict__ partial, long stride, int used,
                                                             int M, double* __restrict__ acc) {
    __shared__ double red[1024];
    double s = 0.0;
    for (long i = threadIdx.x; i < (long)M * used; i += 1024) s += partial[i / used * stride + i % used];
    red[threadIdx.x] = s;
    for (int w = 512; w > 0; w >>= 1) {
        __syncthreads();
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    }
    if (threadIdx.x == 0) acc[0] = red[0];
}

// Label-smoothed cross-entropy over one row of V logits per block.
// q_v = ls / V + (1 - ls) [v == label];  loss_row = -sum_v q_v log p_v
//   = lse - ls / V sum_v z_v - (1 - ls) z_label,   lse = log sum_v exp z_v;
// dZ_v = (p_v - q_v) / norm.
// With clip > 0 every logit first becomes min(max(z, -clip), clip) and the
// gradient passes only where |z| <= clip (the clip's derivative).
// A label outside [0, V) is read as class 0 (so every access stays inside
// the row) and raises bad_label[0], which the host reports.
template <typename T>
__global__ void __launch_bounds__(256) xent_kernel(T* __restrict__ z, int V, const int* __restrict__ labels,
                                                   float ls, float clip, double norm, double* __restrict__ partial,
                                                   int* __restrict__ bad_label) {
    __shared__ float red[4];
    __shared__ float bc[2];
    const long row = blockIdx.x;
    T* zr = z + row * (long)V;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float lim = clip > 0.f ? clip : INFINITY;
    auto logit = [&](int v) { return fminf(fmaxf(to_f32(zr[v]), -lim), lim); };
    float m = -INFINITY, sz = 0.f;
    for (int v = tid; v < V; v += 256) {
        const float x = logit(v);
        m = fmaxf(m, x);
        sz += x;
    }
    m = wave_max(m);
    sz = wave_sum(sz);
    if (lane == 0) red[w] = m;
    __syncthreads();
    if (tid == 0) bc[0] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    m = bc[0];
    __syncthreads();
    if (lane == 0) red[w] = sz;
    __syncthreads();
    if (tid == 0) bc[1] = red[0] + red[1] + red[2] + red[3];
    __syncthreads();
    sz = bc[1];
    float se = 0.f;
    for (int v = tid; v < V; v += 256) se += expf(logit(v) - m);
    se = wave_sum(se);
    __syncthreads();
    if (lane == 0) red[w] = se;
    __syncthreads();
    if (tid == 0) bc[0] = red[0] + red[1] + red[2] + red[3];
    __syncthreads();
    se = bc[0];
    const int raw = labels[row];
    const bool ok = raw >= 0 && raw < V;
    const int lab = ok ? raw : 0;
    if (!ok && tid == 0) bad_label[0] = 1;
    const float zl = logit(lab);
    __syncthreads();
    const float lse = m + logf(se);
    const float inv = 1.f / se, u = ls / V, gn = (float)(1.0 / norm);
    for (int v = tid; v < V; v += 256) {
        const float z = to_f32(zr[v]);
        const float p = expf(fminf(fmaxf(z, -lim), lim) - m) * inv;
        const float q = u + (v == lab ? 1.f - ls : 0.f);
        zr[v] = to_elt<T>(fabsf(z) <= lim ? (p - q) * gn : 0.f);
    }
    if (tid == 0) partial[row] = ((double)lse - (double)u * sz - (1.0 - ls) * zl) / norm;
}

// The same for bf16 logits (V % 8 == 0, V <= 2048 NC) with the row in LDS: read
// once and written once with 16-byte accesses, where the kernel above reads it four
// times in 2-byte accesses.  A thread works on the same logits in the same order as
// there (v = tid + 256 k), its exponentials stay in registers, and the fused
// multiply-adds are those that kernel compiles to, so the results are the same bit
// for bit.  Bound by HBM and the exponentials' vector instructions: at 1024 rows of
// 32000, 131 MB, 26 us at the copy rate and about as much for the latter; 154 us
// before, 63 now (both inside a step, beside other streams).
template <int NC, bool CLIP>
__global__ void __launch_bounds__(256) xent_rows_kernel(bf16* __restrict__ z, int V, const int* __restrict__ labels,
                                                        float ls, float clip, double norm,
                                                        double* __restrict__ partial, int* __restrict__ bad_label) {
    constexpr int K = 8 * NC;
    __shared__ __attribute__((aligned(16))) bf16 zs[NC * 2048];
    __shared__ float red[3][4];
    const long row = blockIdx.x;
    bf16x8* z8 = reinterpret_cast<bf16x8*>(z + row * (long)V);
    bf16x8* s8 = reinterpret_cast<bf16x8*>(zs);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, n8 = V / 8;
    const int kf = V / 256, rest = kf * 256 + tid;  // logits of every thread, and this thread's one beyond them
    const float lim = CLIP ? clip : INFINITY;
    auto logit = [&](int v) {  // no clip: a NaN counts as -inf, as it does between two limits
        const float x = fmaxf((float)zs[v], -lim);
        return CLIP ? fminf(x, lim) : x;
    };
    const int raw = labels[row];
    const bool ok = raw >= 0 && raw < V;
    const int lab = ok ? raw : 0;
    if (!ok && tid == 0) bad_label[0] = 1;
    bf16x8 v[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (tid + 256 * c < n8) v[c] = z8[tid + 256 * c];
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (tid + 256 * c < n8) s8[tid + 256 * c] = v[c];
    __syncthreads();
    const float zl = logit(lab), raw_lab = (float)zs[lab];
    float ex[K], xr = -INFINITY, m = -INFINITY, sz = 0.f, se = 0.f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (256 * k + 255 >= V) break;
        ex[k] = logit(tid + 256 * k);
        m = fmaxf(m, ex[k]);
        sz += ex[k];
    }
    if (rest < V) {
        xr = logit(rest);
        m = fmaxf(m, xr);
        sz += xr;
    }
    m = wave_max(m);
    sz = wave_sum(sz);
    if (lane == 0) {
        red[0][w] = m;
        red[1][w] = sz;
    }
    __syncthreads();  // also: every thread has read the label's logit
    m = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    sz = red[1][0] + red[1][1] + red[1][2] + red[1][3];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (256 * k + 255 >= V) break;
        ex[k] = expf(ex[k] - m);
        se += ex[k];
    }
    if (rest < V) {
        xr = expf(xr - m);
        se += xr;
    }
    se = wave_sum(se);
    if (lane == 0) red[2][w] = se;
    __syncthreads();
    se = red[2][0] + red[2][1] + red[2][2] + red[2][3];
    const float inv = 1.f / se, u = ls / V, gn = (float)(1.0 / norm);
    auto grad = [&](float logit, float e, float q) {
        return (bf16)(fabsf(logit) <= lim ? __builtin_fmaf(e, inv, -q) * gn : 0.f);
    };
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (256 * k + 255 >= V) break;
        const int i = tid + 256 * k;
        zs[i] = grad((float)zs[i], ex[k], u);
    }
    if (rest < V) zs[rest] = grad((float)zs[rest], xr, u);
    if (tid == (lab & 255)) zs[lab] = grad(raw_lab, expf(zl - m), u + (1.f - ls));
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (tid + 256 * c < n8) z8[tid + 256 * c] = s8[tid + 256 * c];
    if (tid == 0) {
        const double lse = m + logf(se);
        partial[row] = __builtin_fma(-(1.0 - ls), (double)zl, __builtin_fma(-(double)u, (double)sz, lse)) / norm;
    }
}

// kn = W, nk = W^T through a 64 x 64 LDS tile (both writes coalesced).
template <typename T>
__global__ void __launch_bounds__(256) refresh_kernel(const float* __restrict__ w, int in, int out,
                                                      T* __restrict__ kn, T* __restrict__ nk) {
    __shared__ float tile[64][65];
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int r = ty; r < 64; r += 4) {
        const int row = r0 + r, col = c0 + tx;
        if (row < in && col < out) {
            const float v = w[(long)row * out + col];
            tile[r][tx] = v;
            kn[(long)row * out + col] = to_elt<T>(v);
        }
    }
    __syncthreads();
    for (int c = ty; c < 64; c += 4) {
        const int col = c0 + c, row = r0 + tx;
        if (row < in && col < out) nk[(long)col * in + row] = to_elt<T>(tile[tx][c]);
    }
}

// Four consecutive elements of a 16-bit working copy, rounded from fp32.
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
template <typename E> struct Copy4;
template <> struct Copy4<bf16> {
    static __device__ __forceinline__ void store(bf16* p, float a, float b, float c, float d) {
        *reinterpret_cast<bf16x4*>(p) = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
    }
};
template <> struct Copy4<_Float16> {
    static __device__ __forceinline__ void store(_Float16* p, float a, float b, float c, float d) {
        *reinterpret_cast<f16x4*>(p) = {(_Float16)a, (_Float16)b, (_Float16)c, (_Float16)d};
    }
};

template <> struct Copy4<float> {
    static __device__ __forceinline__ void store(float* p, float a, float b, float c, float d) {
        *reinterpret_cast<f32x4*>(p) = {a, b, c, d};
    }
};

// The same for bf16 copies of whole 64 x 64 tiles (in, out multiples of 64):
// 16-byte reads of W, 8-byte writes of both copies.  NK: the element type of
// the transposed copy (bf16, or fp16 for a GEMM with fp16 operands).
template <typename NK>
__global__ void __launch_bounds__(256) refresh_bf16_tiles(const float* __restrict__ w, int in, int out,
                                                          bf16* __restrict__ kn, NK* __restrict__ nk) {
    __shared__ float tile[64][65];
    const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int idx = t + 256 * k, r = idx >> 4, c = (idx & 15) * 4;
        const long o = (long)(r0 + r) * out + c0 + c;
        const f32x4 v = *reinterpret_cast<const f32x4*>(w + o);
#pragma unroll
        for (int j = 0; j < 4; ++j) tile[r][c + j] = v[j];
        *reinterpret_cast<bf16x4*>(kn + o) = {(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]};
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int idx = t + 256 * k, c = idx >> 4, r = (idx & 15) * 4;
        Copy4<NK>::store(nk + (long)(c0 + c) * in + r0 + r, tile[r][c], tile[r + 1][c], tile[r + 2][c], tile[r + 3][c]);
    }
}

// W <- W - lr G (SGD), or the RMSProp step (rms: ms <- rho ms + (1 - rho) G^2;
// W <- W - lr G / sqrt(ms + eps)), of one parameter.  Which product goes unrounded
// into its sum is written out, since what the compiler fuses by itself changes with
// the code around: W and ms take fma(-lr, G, W) and fma(rho, ms, (1 - rho) G^2);
// `apart` (see update_kernel): W - (lr G) and fma(1 - rho, G^2, rho ms).
__device__ __forceinline__ float update_one(float w, float g, float& m, float lr, float rho, float eps, int rms,
                                            int apart) {
#pragma clang fp contract(off)
    if (rms) {
        const float gg = g * g, k = 1.f - rho;
        m = apart ? __builtin_fmaf(k, gg, rho * m) : __builtin_fmaf(rho, m, k * gg);
        w -= lr * g / sqrtf(m + eps);
    } else {
        w = apart ? w - lr * g : __builtin_fmaf(-lr, g, w);
    }
    return w;
}

// The update of linears l0 .. l1 - 1 of the table, fused with the refresh of
// their working copies: a workgroup per 64 x 64 tile of W (tiles of the table's
// linears end to end, from linear l0's first) reads W and G once and writes W,
// the copy kn and, through an LDS tile, the transposed copy nk; 16-byte accesses
// where in and out are multiples of 64.  Workgroups from `tiles` on update the
// parameters outside the weights: workgroup tiles + r the float range r, with the
// roundings of `apart` where every linear is whole tiles in bf16 (a kernel of their
// own updated them there, and the results keep its bits).
// Bound by HBM for large layers (16 bytes per weight with SGD, 12 with fp32
// copies); for small ones by the launches, which one per linear, plus one for
// the rest, cost 5 us of host time each: the smallest fp32 step 1085 -> 959 us,
// two ragged layers 1495 -> 1361.
template <typename T>
__global__ void __launch_bounds__(256) update_kernel(float* __restrict__ master, const float* __restrict__ grads,
                                                     float* __restrict__ ms, float lr, float rho, float eps, int rms,
                                                     T* __restrict__ welt, const UpdateLinear* __restrict__ tab, int l0,
                                                     int l1, int tiles, const long* __restrict__ ranges, int apart) {
    __shared__ float tile[64][65];
    const int t = threadIdx.x;
    if ((int)blockIdx.x >= tiles) {
        const long r = blockIdx.x - tiles, off = ranges[2 * r], n = ranges[2 * r + 1];
        for (long i = off + t; i < off + n; i += 256) {
            float m = rms ? ms[i] : 0.f;
            master[i] = update_one(master[i], grads[i], m, lr, rho, eps, rms, apart);
            if (rms) ms[i] = m;
        }
        return;
    }
    const int id = tab[l0].tile0 + blockIdx.x;
    int l = l0;
    for (int hi = l1; l + 1 < hi;) {  // the last linear whose first tile is not after id
        const int mid = (l + hi) / 2;
        if (tab[mid].tile0 <= id)
            l = mid;
        else
            hi = mid;
    }
    const UpdateLinear u = tab[l];
    const int nx = (u.out + 63) / 64, k0 = id - u.tile0, r0 = k0 / nx * 64, c0 = k0 % nx * 64;
    float* w = master + u.w;
    const float* g = grads + u.w;
    float* mm = ms + u.w;
    T* kn = welt + u.kn;
    T* nk = welt + u.nk;
    if (u.in % 64 == 0 && u.out % 64 == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int idx = t + 256 * k, r = idx >> 4, c = (idx & 15) * 4;
            const long o = (long)(r0 + r) * u.out + c0 + c;
            f32x4 v = *reinterpret_cast<const f32x4*>(w + o);
            const f32x4 gv = *reinterpret_cast<const f32x4*>(g + o);
            f32x4 m = {0.f, 0.f, 0.f, 0.f};
            if (rms) m = *reinterpret_cast<const f32x4*>(mm + o);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float me = m[e];
                v[e] = update_one(v[e], gv[e], me, lr, rho, eps, rms, 0);
                m[e] = me;
            }
            if (rms) *reinterpret_cast<f32x4*>(mm + o) = m;
            *reinterpret_cast<f32x4*>(w + o) = v;
#pragma unroll
            for (int j = 0; j < 4; ++j) tile[r][c + j] = v[j];
            Copy4<T>::store(kn + o, v[0], v[1], v[2], v[3]);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int idx = t + 256 * k, c = idx >> 4, r = (idx & 15) * 4;
            const long o = (long)(c0 + c) * u.in + r0 + r;
            if (u.nk16)  // fp16 in place of the partition's 16-bit type
                Copy4<_Float16>::store(reinterpret_cast<_Float16*>(nk) + o, tile[r][c], tile[r + 1][c], tile[r + 2][c],
                                       tile[r + 3][c]);
            else
                Copy4<T>::store(nk + o, tile[r][c], tile[r + 1][c], tile[r + 2][c], tile[r + 3][c]);
        }
        return;
    }
    const int tx = t & 63, ty = t >> 6;
    for (int r = ty; r < 64; r += 4) {
        const int row = r0 + r, col = c0 + tx;
        if (row < u.in && col < u.out) {
            const long o = (long)row * u.out + col;
            float m = rms ? mm[o] : 0.f;
            const float v = update_one(w[o], g[o], m, lr, rho, eps, rms, 0);
            if (rms) mm[o] = m;
            w[o] = v;
            tile[r][tx] = v;
            kn[o] = to_elt<T>(v);
        }
    }
    __syncthreads();
    for (int c = ty; c < 64; c += 4) {
        const int col = c0 + c, row = r0 + tx;
        if (row < u.in && col < u.out) nk[(long)col * u.in + row] = to_elt<T>(tile[tx][c]);
    }
}

// fp4 copy of bf16 rows (the W^T working copy, rows of `in` values): one wave
// per row; 8 values per lane step; one E8M0 scale per row (see e2m1_code).
__global__ void __launch_bounds__(256) quant4_rows_kernel(const bf16* __restrict__ src, int rows, int in,
                                                          unsigned char* __restrict__ q4, unsigned char* __restrict__ sc) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const bf16x8* r8 = reinterpret_cast<const bf16x8*>(src + row * in);
    const int n8 = in / 8;
    float amax = 0.f;
    for (int i = lane; i < n8; i += 64) {
        const bf16x8 v = r8[i];
#pragma unroll
        for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf((float)v[e]));
    }
    const unsigned s = e8m0_for_amax(wave_max(amax));
    const float inv = e8m0_inv(s);
    unsigned* o4 = reinterpret_cast<unsigned*>(q4 + row * (in / 2));
    for (int i = lane; i < n8; i += 64) {
        const bf16x8 v = r8[i];
        unsigned q = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) q |= e2m1_code((float)v[e] * inv) << (4 * e);
        o4[i] = q;
    }
    if (lane == 0) sc[row] = (unsigned char)s;
}

// MFMA-loop peak probe: 4 waves per workgroup, each with 8 independent
// 32x32 accumulators and two operand sets of pseudo-random bf16 (so that the
// multiplier inputs toggle as in a real GEMM); 16 MFMAs per trip.
__global__ void __launch_bounds__(256) mfma_peak_kernel(float* __restrict__ out, int iters) {
    typedef __bf16 b8 __attribute__((ext_vector_type(8)));
    typedef float f16v __attribute__((ext_vector_type(16)));
    unsigned h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
    b8 a[2], b[2];
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h = h * 1664525u + 1013904223u;
            a[k][e] = (__bf16)(((int)(h >> 16) - 32768) * (1.f / 32768.f));
            h = h * 1664525u + 1013904223u;
            b[k][e] = (__bf16)(((int)(h >> 16) - 32768) * (1.f / 32768.f));
        }
    f16v c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) c[j][r] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int j = 0; j < 8; ++j) c[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[k], b[k], c[j], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += c[j][r];
    out[blockIdx.x * 256 + threadIdx.x] = s;
}

__global__ void __launch_bounds__(256) finite_kernel(const float* __restrict__ x, long count, int* __restrict__ flag) {
    bool bad = false;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < count; i += (long)gridDim.x * 256)
        bad |= !isfinite(x[i]);
    if (__any(bad) && (threadIdx.x & 63) == 0) flag[0] = 1;
}

int ew_grid(long count) {
    long g = (count + 255) / 256;
    return (int)(g < EW_BLOCKS ? (g > 0 ? g : 1) : EW_BLOCKS);
}

} // namespace

int loss_blocks() { return LOSS_BLOCKS; }
int xent_partials(long rows) { return (int)rows; }

gp_status intake(int dtype, const void* src, void* stash, float* x32, long count, hipStream_t st) {
    auto a16 = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    if (dtype == GP_BF16 && count % 8 == 0 && a16(src) && a16(stash) && a16(x32)) {
        klaunch(intake_bf16_v8, ew_grid(count / 8), 256, 0, st, reinterpret_cast<const bf16x8*>(src),
                reinterpret_cast<bf16x8*>(stash), reinterpret_cast<f32x4*>(x32), count / 8);
    } else if (dtype == GP_BF16)
        klaunch(intake_kernel<bf16>, ew_grid(count), 256, 0, st, reinterpret_cast<const bf16*>(src),
                                                             reinterpret_cast<bf16*>(stash), x32, count);
    else
        klaunch(intake_kernel<float>, ew_grid(count), 256, 0, st, reinterpret_cast<const float*>(src),
                                                              reinterpret_cast<float*>(stash), x32, count);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status cast_out(int dtype, const float* src, void* dst, long count, hipStream_t st) {
    if (dtype == GP_BF16) klaunch(cast_kernel<bf16>, ew_grid(count), 256, 0, st, src, reinterpret_cast<bf16*>(dst), count);
    else klaunch(cast_kernel<float>, ew_grid(count), 256, 0, st, src, reinterpret_cast<float*>(dst), count);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status mse_grad(int dtype, const float* y, const void* target, long count, double norm, float* d32, void* delt,
                   double* partial, int* nblk, hipStream_t st) {
    *nblk = LOSS_BLOCKS;
    if (count % 4) return set_error(GP_ERR_INVALID_ARG, "mse: element count must be a multiple of 4");
    const int tvec = (reinterpret_cast<uintptr_t>(target) & (dtype == GP_BF16 ? 7 : 15)) == 0;
    if (dtype == GP_BF16)
        klaunch(mse_kernel<bf16>, LOSS_BLOCKS, 256, 0, st, y, reinterpret_cast<const bf16*>(target), count, norm, d32,
                                                      reinterpret_cast<bf16*>(delt), partial, tvec);
    else
        klaunch(mse_kernel<float>, LOSS_BLOCKS, 256, 0, st, y, reinterpret_cast<const float*>(target), count, norm, d32,
                                                       reinterpret_cast<float*>(delt), partial, tvec);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status loss_finalize(const double* partial, long stride, int used, int M, double* acc, hipStream_t st) {
    klaunch(loss_finalize_kernel, 1, 1024, 0, st, partial, stride, used, M, acc);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status xent_ls(int dtype, void* z, long rows, int V, const int* labels, float ls, float clip, double norm,
                  double* partial, int* bad_label, hipStream_t st) {
    if (dtype == GP_BF16 && V % 8 == 0 && V <= 16 * 2048) {
        bf16* zb = reinterpret_cast<bf16*>(z);
        const int nc = (V + 2047) / 2048;
#define GP_XENT(NC)                                                                                                  \
    do {                                                                                                             \
        if (clip > 0.f)                                                                                              \
            klaunch(xent_rows_kernel<NC, true>, (unsigned)rows, 256, 0, st, zb, V, labels, ls, clip, norm, partial,  \
                    bad_label);                                                                                      \
        else                                                                                                         \
            klaunch(xent_rows_kernel<NC, false>, (unsigned)rows, 256, 0, st, zb, V, labels, ls, clip, norm, partial, \
                    bad_label);                                                                                      \
    } while (0)
        if (nc <= 1)
            GP_XENT(1);
        else if (nc <= 2)
            GP_XENT(2);
        else if (nc <= 4)
            GP_XENT(4);
        else if (nc <= 8)
            GP_XENT(8);
        else
            GP_XENT(16);
#undef GP_XENT
    } else if (dtype == GP_BF16)
        klaunch(xent_kernel<bf16>, (unsigned)rows, 256, 0, st, reinterpret_cast<bf16*>(z), V, labels, ls, clip, norm,
                partial, bad_label);
    else
        klaunch(xent_kernel<float>, (unsigned)rows, 256, 0, st, reinterpret_cast<float*>(z), V, labels, ls, clip, norm,
                partial, bad_label);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status mfma_peak(hipStream_t st, double* tflops) {
    int dev = 0, cus = 0;
    GP_HIP(hipGetDevice(&dev));
    GP_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    const int grid = 2 * cus, iters = 2000;
    float* out = nullptr;
    GP_HIP(hipMalloc(reinterpret_cast<void**>(&out), (size_t)grid * 256 * sizeof(float)));
    hipEvent_t e0 = nullptr, e1 = nullptr;
    gp_status s = GP_OK;
    double best = 0.0;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) s = set_error(GP_ERR_HIP, "mfma_peak: event");
    for (int rep = 0; rep < 4 && s == GP_OK; ++rep) {
        hipEventRecord(e0, st);
        klaunch(mfma_peak_kernel, grid, 256, 0, st, out, iters);
        const hipError_t le = take_launch_status();
        hipEventRecord(e1, st);
        float ms = 0.f;
        if (le != hipSuccess || hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            s = set_error(GP_ERR_HIP, "mfma_peak: launch or timing failed");
            break;
        }
        const double fl = (double)grid * 4 * iters * 16 * 32768.0;
        if (rep > 0 && ms > 0.f) best = std::max(best, fl / (ms * 1e-3) * 1e-12);  // the first run warms up
    }
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
    hipStreamSynchronize(st);
    hipFree(out);
    if (s == GP_OK && tflops) *tflops = best;
    return s;
}

gp_status update_linears(int dtype, float* master, const float* grads, float* ms, float lr, float rho, float eps,
                         void* welt, const UpdateLinear* table, int l0, int l1, int tiles, const long* ranges,
                         int nranges, int apart, hipStream_t st) {
    if (tiles + nranges <= 0) return GP_OK;
    if (dtype == GP_BF16)
        klaunch(update_kernel<bf16>, tiles + nranges, 256, 0, st, master, grads, ms, lr, rho, eps, ms ? 1 : 0,
                static_cast<bf16*>(welt), table, l0, l1, tiles, ranges, apart);
    else
        klaunch(update_kernel<float>, tiles + nranges, 256, 0, st, master, grads, ms, lr, rho, eps, ms ? 1 : 0,
                static_cast<float*>(welt), table, l0, l1, tiles, ranges, apart);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status quantize_rows_fp4(const void* nk, int out, int in, void* q4, void* q4s, hipStream_t st) {
    if (in % 8) return set_error(GP_ERR_UNSUPPORTED, "refresh: fp4 copies are made from bf16 rows");
    klaunch(quant4_rows_kernel, (out + 3) / 4, 256, 0, st, reinterpret_cast<const bf16*>(nk), out, in,
            static_cast<unsigned char*>(q4), static_cast<unsigned char*>(q4s));
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status refresh_linear(int dtype, const float* w, int in, int out, void* kn, void* nk, void* q4, void* q4s,
                         hipStream_t st, bool nk16) {
    dim3 grid((out + 63) / 64, (in + 63) / 64);
    if (nk16 && (dtype != GP_BF16 || in % 64 || out % 64 || q4))
        return set_error(GP_ERR_INVALID_ARG, "refresh: an fp16 W^T needs bf16 whole 64 x 64 tiles and no fp4 copy");
    if (nk16)
        klaunch(refresh_bf16_tiles<_Float16>, grid, 256, 0, st, w, in, out, reinterpret_cast<bf16*>(kn),
                reinterpret_cast<_Float16*>(nk));
    else if (dtype == GP_BF16 && in % 64 == 0 && out % 64 == 0)
        klaunch(refresh_bf16_tiles<bf16>, grid, 256, 0, st, w, in, out, reinterpret_cast<bf16*>(kn),
                reinterpret_cast<bf16*>(nk));
    else if (dtype == GP_BF16)
        klaunch(refresh_kernel<bf16>, grid, 256, 0, st, w, in, out, reinterpret_cast<bf16*>(kn), reinterpret_cast<bf16*>(nk));
    else
        klaunch(refresh_kernel<float>, grid, 256, 0, st, w, in, out, reinterpret_cast<float*>(kn), reinterpret_cast<float*>(nk));
    GP_LAUNCH_CHECK();
    if (q4) {
        if (dtype != GP_BF16) return set_error(GP_ERR_UNSUPPORTED, "refresh: fp4 copies are made from bf16 rows");
        return quantize_rows_fp4(nk, out, in, q4, q4s, st);
    }
    return GP_OK;
}

// All-ones bytes over [p, p + bytes): a NaN in every fp32, bf16 and fp64
// element.  16-byte stores over the aligned middle, byte stores at the edges.
__global__ void __launch_bounds__(256) poison_kernel(unsigned char* __restrict__ p, long head, long n16, long tail) {
    const long t = (long)blockIdx.x * 256 + threadIdx.x, stride = (long)gridDim.x * 256;
    if (t < head) p[t] = 0xFF;
    uint4* q = reinterpret_cast<uint4*>(p + head);
    for (long i = t; i < n16; i += stride) q[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (t < tail) p[head + 16 * n16 + t] = 0xFF;
}

gp_status poison_fill(void* p, size_t bytes, hipStream_t st) {
    if (!p || bytes == 0) return GP_OK;
    unsigned char* c = static_cast<unsigned char*>(p);
    const long head = (long)((16 - (reinterpret_cast<uintptr_t>(c) & 15)) & 15);
    const long h = head < (long)bytes ? head : (long)bytes;
    const long n16 = ((long)bytes - h) / 16, tail = (long)bytes - h - 16 * n16;
    klaunch(poison_kernel, ew_grid(n16 > 256 ? n16 : 256), 256, 0, st, c, h, n16, tail);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

// Empty kernel that delimits a timed launch in a profiler's dispatch list.
// Its grid encodes the label (role workgroups in x, edge + 1 in y), which a
// kernel trace records.
__global__ void role_marker_kernel() {}

gp_status role_marker(int role, int edge, hipStream_t st) {
    klaunch(role_marker_kernel, dim3(role, edge + 1), 64, 0, st);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

gp_status finite_check(const float* x, long count, int* flag, hipStream_t st) {
    klaunch(finite_kernel, ew_grid(count), 256, 0, st, x, count, flag);
    GP_LAUNCH_CHECK();
    return GP_OK;
}

} // namespace gp
