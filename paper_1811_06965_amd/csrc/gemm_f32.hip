// gemm_f32.hip -- fp32 GEMM of fp32 partitions on the matrix cores.
//
//   C[m, n] = sum_k A(m, k) B(n, k), then the fused epilogues of gemm.hip.
//
// The fp32 MFMAs run at a sixteenth of the bf16 rate (157 TFLOP/s on the chip),
// so HBM and L2 traffic is never the limit.  What bounds these GEMMs is how
// many SIMDs have an output block and how long one block's serial k-chain is.
// Both MFMA shapes add their k products one after the other, each rounded (an
// fma chain in k order), so a 16 x 16 x 4 step gives bit for bit what two
// 32 x 32 x 2 steps give, in a quarter of the time per k.  Small problems
// therefore take 32 x 32 tiles of four waves with one 16 x 16 block each (512 x
// 512 outputs already give every CU a workgroup), larger ones 64 x 64 and 128 x
// 64 tiles with 32 x 32 blocks per wave.  Every tile sums each element in the
// same order (k-tiles of 32; within 16 k: 0 8 1 9 2 10 .. 7 15), so the result
// depends on neither the tile nor the number of rows.
//
// Tiles are copied global -> LDS with buffer_load_dwordx4 ... lds into a ring
// of NS stages of 32 k, one barrier per k-tile, explicit vmcnt waits (as in
// gemm_dl).  The last k-tile of a K that is no multiple of 32 loads zeros
// beyond K (per-lane offsets out of the buffer's range), so any K the operand
// layout allows takes this path.
#include <algorithm>

#include "gemm_tile.hpp"
#include "kernels.hpp"

namespace gp {

namespace {

__device__ __forceinline__ float bload_f32(Rsrc r, uint32_t off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void bstore_f32(Rsrc r, uint32_t off, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, off, 0, 0);
}

// Epilogue of NR accumulator registers of one column: register r is row
// row0 + 8 (r / 4) + r % 4.  The loads are issued before any store.
template <int EPI, int NR>
__device__ __forceinline__ void epilogue_col(const GemmArgs& a, const float (&v)[NR], int row0, int col) {
    const Rsrc c = make_rsrc(a.C, (uint32_t)(((long)(a.M - 1) * a.ldc + a.N) * 4));
    float in[NR];
    uint32_t oc[NR];
    Rsrc aux;
    if constexpr (EPI == EPI_RES_F32 || EPI == EPI_RELU_MASK)
        aux = make_rsrc(a.aux, (uint32_t)(((long)(a.M - 1) * a.ldaux + a.N) * 4));
    const bool colok = col < a.N;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int row = row0 + (r >> 2) * 8 + (r & 3);
        const bool ok = colok && row < a.M;
        oc[r] = ok ? (uint32_t)(((long)row * a.ldc + col) * 4) : OOB;
        if constexpr (EPI == EPI_RES_F32 || EPI == EPI_RELU_MASK)
            in[r] = bload_f32(aux, ok ? (uint32_t)(((long)row * a.ldaux + col) * 4) : OOB);
        else if constexpr (EPI == EPI_ACC_F32)
            in[r] = a.accumulate ? bload_f32(c, oc[r]) : 0.f;
    }
    float bv = 0.f;
    if constexpr (EPI == EPI_STORE || EPI == EPI_RES_F32) bv = a.bias && colok ? a.bias[col] : 0.f;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        float x = v[r];
        if constexpr (EPI == EPI_STORE) {
            x += bv;
            if (a.relu) x = fmaxf(x, 0.f);
        } else if constexpr (EPI == EPI_RES_F32) {
            x += in[r] + bv;
        } else if constexpr (EPI == EPI_RELU_MASK) {
            x = in[r] > 0.f ? x : 0.f;
        } else if constexpr (EPI == EPI_ACC_F32) {
            x += in[r];
        }
        bstore_f32(c, oc[r], x);
        if constexpr (EPI == EPI_RES_F32) {
            const int row = row0 + (r >> 2) * 8 + (r & 3);
            if (a.C2) {
                const Rsrc c2 = make_rsrc(a.C2, (uint32_t)(((long)(a.M - 1) * a.ldc2 + a.N) * 4));
                bstore_f32(c2, oc[r] != OOB ? (uint32_t)(((long)row * a.ldc2 + col) * 4) : OOB, x);
            }
        }
    }
}

// k (within a k-tile) of the 16 bytes this lane loads in 1 KB block `blk` of an
// operand of `width` rows.
template <bool KM>
__device__ __forceinline__ int k_of(int blk, int width, int lane) {
    if constexpr (KM)
        return ((lane & 7) ^ swz(blk * 8 + (lane >> 3))) * 4;
    else
        return (blk * 1024 + 16 * lane) / (4 * width);
}
// m (within the tile) of those 16 bytes, m-contiguous operands (see frag).
__device__ __forceinline__ int m_of(int blk, int width, int lane) {
    return ((blk * 1024 + 16 * lane) % (4 * width) / 4) ^ (((k_of<false>(blk, width, lane) >> 3) & 1) << 4);
}
template <int P, bool KM>
__device__ __forceinline__ void mask_beyond(uint32_t* vo, int blk0, int width, int krem, int lane) {
#pragma unroll
    for (int i = 0; i < P; ++i)
        if (k_of<KM>(blk0 + i, width, lane) >= krem) vo[i] = OOB;
}
template <int P>
__device__ __forceinline__ void load_blocks(Rsrc g, const uint32_t* vo, int so, char* dst) {
#pragma unroll
    for (int i = 0; i < P; ++i) __builtin_amdgcn_raw_ptr_buffer_load_lds(g, (LdsPtr)(dst + i * 1024), 16, vo[i], so, 0, 0);
}

// A k-tile is KS steps of four MFMAs.  With j = lane / 16 (BLK = 16) or h =
// lane / 32 (BLK = 32) the lane supplies, to MFMA i of step s,
//   BLK = 32 (KS = 4): k = 16 (s / 2) + 4 (s % 2) + i + 8 h
//   BLK = 16 (KS = 2): k = 16 s + 2 i + j / 2 + 8 (j % 2)
template <int BLK> struct Block;
template <> struct Block<32> {
    typedef f32x16 Acc;
    static constexpr int NR = 16, KS = 4;  // accumulator registers; steps per k-tile
    static __device__ __forceinline__ int row_of(int lane) { return 4 * (lane >> 5); }
    static __device__ __forceinline__ int k_hi(int lane) { return lane >> 5; }
    static __device__ __forceinline__ int k_of(int step, int i, int lane) {
        return 16 * (step >> 1) + 4 * (step & 1) + i + 8 * k_hi(lane);
    }
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int chunk(int step, int lane) {
        return 4 * (step >> 1) + 2 * k_hi(lane) + (step & 1);
    }
    static __device__ __forceinline__ void pick(f32x4 v, float* f) {
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = v[e];
    }
};
template <> struct Block<16> {
    typedef f32x4 Acc;
    static constexpr int NR = 4, KS = 2;
    static __device__ __forceinline__ int row_of(int lane) { return 4 * (lane >> 4); }
    static __device__ __forceinline__ int k_hi(int lane) { return (lane >> 4) & 1; }
    static __device__ __forceinline__ int k_of(int step, int i, int lane) {
        return 16 * step + 2 * i + (lane >> 5) + 8 * k_hi(lane);
    }
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // Lanes l and l + 32 read the first and second four of the eight k they
    // share, (k, k+1, k+2, k+3) and (k+4, ..); swapping the upper half of one
    // register with the lower half of the next leaves k | k+1 in one and
    // k+4 | k+5 in the other.
    static __device__ __forceinline__ int chunk(int step, int lane) { return 4 * step + 2 * k_hi(lane) + (lane >> 5); }
    static __device__ __forceinline__ void pick(f32x4 v, float* f) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2 * e]), __float_as_uint(v[2 * e + 1]),
                                                            false, false);
            f[e] = __uint_as_float(r[0]);
            f[e + 2] = __uint_as_float(r[1]);
        }
#endif
    }
};

// A lane's operands of one step from an LDS tile.  KM: rows of 32 k (128
// bytes) per m, 16-byte chunks XOR-swizzled by swz(row); one 16-byte read.
// !KM: 32 k-rows of `width` consecutive m, where k-rows 8 .. 15 of every 16
// have m's bit 4 flipped (with BLK = 16 a half-wave reads k and k + 8 at once:
// otherwise the same 16 banks); dword reads.
template <int BLK, bool KM>
__device__ __forceinline__ void frag(const char* s, int row, int width, int step, int lane, float* f) {
    typedef Block<BLK> B;
    if constexpr (KM) {
        B::pick(*reinterpret_cast<const f32x4*>(s + row * 128 + ((B::chunk(step, lane) ^ swz(row)) << 4)), f);
    } else {
        const char* p = s + (row ^ (B::k_hi(lane) << 4)) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = *reinterpret_cast<const float*>(p + B::k_of(step, i, lane) * width * 4);
    }
}

// Add this thread's column-sum shares of one k-tile (share idx: column idx %
// BN, k-rows 4 (idx / BN) .. + 3).
template <int BM, int BN, int CPT>
__device__ __forceinline__ void add_colsum(const char* stage, int tid, int nt, float* cs) {
#pragma unroll
    for (int p = 0; p < CPT; ++p) {
        const int idx = p * nt + tid, col = idx % BN, kb = idx / BN;
        const float* b = reinterpret_cast<const float*>(stage + BM * 128) + 4 * kb * BN + (col ^ (((kb >> 1) & 1) << 4));
#pragma unroll
        for (int q = 0; q < 4; ++q) cs[p] += b[q * BN];
    }
}

// KM: both operands k-contiguous (A[m lda + k], B[n ldb + k]); !KM: both
// m/n-contiguous (A[k lda + m], B[k ldb + n]).  WM x WN waves, each (BM / WM) x
// (BN / WN) outputs in BLK x BLK blocks.
template <int BM, int BN, int WM, int WN, int BLK, int NS, int EPI, bool KM>
__global__ void __launch_bounds__(64 * WM * WN) gemm_f32_kernel(GemmArgs args) {
    constexpr int BK = 32;  // k per stage
    constexpr int NW = WM * WN;
    typedef Block<BLK> Bk;
    constexpr int TM = BM / WM / BLK, TN = BN / WN / BLK, NR = Bk::NR, KS = Bk::KS;
    constexpr int STAGE = (BM + BN) * 128;
    constexpr int PA = BM / (8 * NW), PB = BN / (8 * NW), LPW = PA + PB;  // 1 KB load blocks per wave
    static_assert(PA * 8 * NW == BM && PB * 8 * NW == BN, "load blocks");
    constexpr bool COLSUM = !KM && EPI == EPI_ACC_F32;
    constexpr int CPT = BN * 8 / (64 * NW);  // column-sum shares per thread (8 per column)
    static_assert(!COLSUM || CPT * 64 * NW == BN * 8, "column sums");
    // one LDS object only: with a second one the compiler waits for every
    // outstanding direct-to-LDS load (vmcnt(0)) before each LDS read
    __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];
    static_assert(NS >= 2 && NS * STAGE <= 160 * 1024 && BN * 8 * 4 <= NS * STAGE, "LDS");

    const int tid = threadIdx.x, lane = tid & 63, wave = uniform_wave_id(tid);
    const int wm = wave / WN, wn = wave % WN, fr = lane & (BLK - 1);
    int tm, tn;
    band_tile(xcd_order(blockIdx.x, gridDim.x), (args.M + BM - 1) / BM, (args.N + BN - 1) / BN, 8, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int K = args.K, nk = (K + BK - 1) / BK;

    Rsrc A, B;
    uint32_t voa[PA], vob[PB];
    int ka, kb;  // bytes per k-tile advance
    if constexpr (KM) {
        A = make_rsrc(args.A, (uint32_t)(((long)(args.M - 1) * args.lda + K) * 4));
        B = make_rsrc(args.B, (uint32_t)(((long)(args.N - 1) * args.ldb + K) * 4));
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int row = m0 + (wave * PA + i) * 8 + (lane >> 3);
            voa[i] = row < args.M ? (uint32_t)(((long)row * args.lda + k_of<KM>(wave * PA + i, BM, lane)) * 4) : OOB;
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int row = n0 + (wave * PB + i) * 8 + (lane >> 3);
            vob[i] = row < args.N ? (uint32_t)(((long)row * args.ldb + k_of<KM>(wave * PB + i, BN, lane)) * 4) : OOB;
        }
        ka = kb = BK * 4;
    } else {
        A = make_rsrc(args.A, (uint32_t)(((long)(K - 1) * args.lda + args.M) * 4));
        B = make_rsrc(args.B, (uint32_t)(((long)(K - 1) * args.ldb + args.N) * 4));
#pragma unroll
        for (int i = 0; i < PA; ++i) {
            const int m = m0 + m_of(wave * PA + i, BM, lane);
            voa[i] = m < args.M ? (uint32_t)(((long)k_of<KM>(wave * PA + i, BM, lane) * args.lda + m) * 4) : OOB;
        }
#pragma unroll
        for (int i = 0; i < PB; ++i) {
            const int n = n0 + m_of(wave * PB + i, BN, lane);
            vob[i] = n < args.N ? (uint32_t)(((long)k_of<KM>(wave * PB + i, BN, lane) * args.ldb + n) * 4) : OOB;
        }
        ka = (int)(BK * args.lda * 4);
        kb = (int)(BK * args.ldb * 4);
    }
    const int krem = K - (nk - 1) * BK;  // k of the last tile
#define GP_F32_LOADS(t, st)                                                                   \
    do {                                                                                      \
        load_blocks<PA>(A, voa, (t) * ka, (st) + wave * PA * 1024);                           \
        load_blocks<PB>(B, vob, (t) * kb, (st) + BM * 128 + wave * PB * 1024);                \
    } while (0)
// Issue k-tile t into stage st; on the ragged last tile (no load follows it)
// the lanes beyond K first move out of range and load zeros.
#define GP_F32_ISSUE(t, st)                                                                   \
    do {                                                                                      \
        if ((t) == nk - 1 && krem < BK) {                                                     \
            mask_beyond<PA, KM>(voa, wave * PA, BM, krem, lane);                              \
            mask_beyond<PB, KM>(vob, wave * PB, BN, krem, lane);                              \
        }                                                                                     \
        GP_F32_LOADS(t, st);                                                                  \
    } while (0)

    typename Bk::Acc acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < NR; ++r) acc[i][j][r] = 0.f;
    // Fused bias gradient: the workgroups of the first M tile see every k of
    // their columns.  A column has eight shares, k-rows 4 kb .. 4 kb + 3 of
    // every k-tile each, summed in k order and then in kb order.
    const bool do_colsum = COLSUM && args.colsum != nullptr && tm == 0;
    float cs[COLSUM ? CPT : 1] = {};

    const int ar = wm * (BM / WM) + fr, br = wn * (BN / WN) + fr;
    // The fragments of the next step are read while the current one is
    // multiplied (reading a whole tile ahead was no faster); on a tile's last
    // step the next tile must have landed, every wave is past its reads of
    // tile t, and t's stage takes tile t + NS.
    float fa[2][TM][4], fb[2][TN][4];
#define GP_F32_FRAGS(slot, st, q)                                                                      \
    do {                                                                                               \
        _Pragma("unroll") for (int i = 0; i < TM; ++i) frag<BLK, KM>((st), ar + i * BLK, BM, (q), lane, fa[slot][i]);  \
        _Pragma("unroll") for (int j = 0; j < TN; ++j)                                                 \
            frag<BLK, KM>((st) + BM * 128, br + j * BLK, BN, (q), lane, fb[slot][j]);                  \
    } while (0)
// One k-tile: waits (WAIT), refills its stage (REFILL) and reads ahead.  The
// lgkmcnt(0) of the barrier is repeated in a form the compiler sees, so that
// it does not wait for the read-ahead before multiplying.
#define GP_F32_TILE(cst, nst, WAIT, REFILL)                                                            \
    do {                                                                                               \
        if constexpr (COLSUM)                                                                          \
            if (do_colsum) add_colsum<BM, BN, CPT>(cst, tid, 64 * NW, cs);                             \
        _Pragma("unroll") for (int q = 0; q < KS; ++q) {                                               \
            const int cur = q & 1;                                                                     \
            if (q + 1 < KS) {                                                                          \
                GP_F32_FRAGS(cur ^ 1, cst, q + 1);                                                     \
            } else {                                                                                   \
                WAIT;                                                                                  \
                lds_barrier();                                                                         \
                __builtin_amdgcn_s_waitcnt(0xC07F);                                                    \
                REFILL;                                                                                \
                GP_F32_FRAGS(cur ^ 1, nst, 0);                                                         \
            }                                                                                          \
            __builtin_amdgcn_sched_barrier(0);                                                         \
            _Pragma("unroll") for (int e = 0; e < 4; ++e)                                              \
                _Pragma("unroll") for (int i = 0; i < TM; ++i)                                         \
                    _Pragma("unroll") for (int j = 0; j < TN; ++j) acc[i][j] =                         \
                        Bk::mma(fa[cur][i][e], fb[cur][j][e], acc[i][j]);                              \
        }                                                                                              \
    } while (0)
#pragma unroll
    for (int p = 0; p < NS; ++p)
        if (p < nk) GP_F32_ISSUE(p, smem + p * STAGE);
    if (nk >= NS)
        wait_vmcnt<(NS - 1) * LPW>();
    else
        wait_vmcnt<0>();
    lds_barrier();
    GP_F32_FRAGS(0, smem, 0);
    // main loop: every tile refills its stage with a whole tile
    int t0 = 0;
    for (; t0 + NS - 1 + NS < nk - 1; t0 += NS) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            char* const cst = smem + (u % NS) * STAGE;
            GP_F32_TILE(cst, smem + ((u + 1) % NS) * STAGE, wait_vmcnt<(NS - 2) * LPW>(),
                        GP_F32_LOADS(t0 + u + NS, cst));
        }
    }
    // the last tiles (at most NS + NS)
    for (; t0 < nk; t0 += NS) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int t = t0 + u;
            if (t >= nk) break;
            char* const cst = smem + (u % NS) * STAGE;
            GP_F32_TILE(cst, smem + ((u + 1) % NS) * STAGE,
                        if (t + NS - 1 < nk) wait_vmcnt<(NS - 2) * LPW>(); else wait_vmcnt<0>(),
                        if (t + NS < nk) GP_F32_ISSUE(t + NS, cst));
        }
    }

#undef GP_F32_TILE
#undef GP_F32_FRAGS
#undef GP_F32_ISSUE
#undef GP_F32_LOADS
    if constexpr (COLSUM) {
        if (do_colsum) {
            // the ring is idle: every load was waited for
            float* red = reinterpret_cast<float*>(smem);  // [8][BN]
            lds_barrier();
#pragma unroll
            for (int p = 0; p < CPT; ++p) red[p * 64 * NW + tid] = cs[p];
            lds_barrier();
            const int col = n0 + tid;
            if (tid < BN && col < args.N) {
                float s = 0.f;
#pragma unroll
                for (int kb = 0; kb < 8; ++kb) s += red[kb * BN + tid];
                args.colsum[col] = args.accumulate ? args.colsum[col] + s : s;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float v[NR];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const float x = acc[i][j][r];
                v[r] = x;
            }
            epilogue_col<EPI, NR>(args, v, m0 + wm * (BM / WM) + i * BLK + Bk::row_of(lane), n0 + br + j * BLK);
        }
}

template <int BM, int BN, int WM, int WN, int BLK, int NS>
gp_status launch(const GemmArgs& a, int epi, bool km, hipStream_t st) {
    const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    constexpr int NT = 64 * WM * WN;
    if (!km) {
        if (epi != EPI_ACC_F32) return set_error(GP_ERR_INVALID_ARG, "gemm: epilogue not instantiated for m-contiguous operands");
        klaunch(gemm_f32_kernel<BM, BN, WM, WN, BLK, NS, EPI_ACC_F32, false>, tiles, NT, 0, st, a);
    } else {
        switch (epi) {
        case EPI_STORE: klaunch(gemm_f32_kernel<BM, BN, WM, WN, BLK, NS, EPI_STORE, true>, tiles, NT, 0, st, a); break;
        case EPI_RES_F32: klaunch(gemm_f32_kernel<BM, BN, WM, WN, BLK, NS, EPI_RES_F32, true>, tiles, NT, 0, st, a); break;
        case EPI_F32: klaunch(gemm_f32_kernel<BM, BN, WM, WN, BLK, NS, EPI_F32, true>, tiles, NT, 0, st, a); break;
        case EPI_RELU_MASK: klaunch(gemm_f32_kernel<BM, BN, WM, WN, BLK, NS, EPI_RELU_MASK, true>, tiles, NT, 0, st, a); break;
        case EPI_ACC_F32: klaunch(gemm_f32_kernel<BM, BN, WM, WN, BLK, NS, EPI_ACC_F32, true>, tiles, NT, 0, st, a); break;
        default: return set_error(GP_ERR_INVALID_ARG, "gemm: unknown epilogue");
        }
    }
    GP_LAUNCH_CHECK();
    return GP_OK;
}

} // namespace

// GemmArgs::force_cfg values of the fp32 tiles (the lower ones are bf16 tiles
// and leave the choice to the rule)
constexpr int F32_TILE0 = 32;

// Tile choice: rounds over the 256 CUs times the time of a tile (measured, us
// per 1024 k): 32 x 32 6.1, 64 x 64 19, 128 x 64 37.5, so the larger tiles are
// taken where they fill their rounds.  A 32 x 32 tile's own chain takes 8.5 us
// per 1024 k, however few there are.  Against the one 128 x 128 register-staged
// tile this replaced (alone, us): 64 x 192 x 64 3.3 from 9.9; 512 x 512 x 2048
// 19.0 from 148; 512 x 2048 x 512 13.0 from 42; weight gradient 512 x 512 x
// 1024 10.4 from 79; 4096 x 8192 x 1024 549 from 552 (125 TFLOP/s of 157).
gp_status gemm_f32(const GemmArgs& a, int epi, bool km, hipStream_t st) {
    auto rounds = [&](long bm, long bn) { return (((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn) + 255) / 256; };
    int cfg = a.force_cfg - F32_TILE0;
    if (cfg < 0) {
        const double t32 = std::max(8.5, 6.1 * rounds(32, 32)), t64 = 19.0 * rounds(64, 64), t128 = 37.5 * rounds(128, 64);
        cfg = t128 <= t64 && t128 <= t32 ? 2 : t64 <= t32 ? 1 : 0;
    }
    switch (cfg) {
    case 0: return launch<32, 32, 2, 2, 16, 4>(a, epi, km, st);
    case 1: return launch<64, 64, 2, 2, 32, 3>(a, epi, km, st);
    default: return launch<128, 64, 4, 2, 32, 3>(a, epi, km, st);
    }
}

} // namespace gp
