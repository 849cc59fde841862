// Dense products on the gfx950 matrix cores: C[M x N] (+)= op(A) op(B), fp32 accumulation.
//
// A workgroup of four 64-wide waves (2 x 2) owns a BM x BN tile of C.  Operand tiles of depth
// BK = 16 are staged through LDS in k-major order (As[k][i], Bs[k][j]) so that the operands of
// v_mfma_f32_32x32x2_f32 (lane l supplies A[i = l%32][k = l/32] and B[k = l/32][j = l%32]) are read
// from consecutive LDS words.  Global loads of the next tile are issued before the MFMAs of the
// current one (register prefetch + two LDS buffers, one barrier per k-step).  bf16 operands are
// widened to fp32 while they are staged.  The vertex-dimension reduction of the weight gradient
// (trans_a) is split over workgroups; partial tiles go to the workspace and are summed in a fixed
// order by a second kernel, which also applies the epilogue.  Small products, narrow or long reductions over vertices and
// products of many rows have kernels of their own below, most of which read their operands straight into registers.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace capgnn {

typedef float floatx16 __attribute__((ext_vector_type(16)));

struct GemmArgs {
    int64_t M, N, K;
    const char *A; int64_t lda;
    const char *B; int64_t ldb;
    char *C; int64_t ldc;           // final destination
    float *part;                    // split partials [S][M][N] or null
    float *colpart;                 // [S][N] column sums of B over the split's k (reductions over vertices), or null
    int64_t k_chunk;                // reduction range per grid.z
    int a_vec, b_vec;               // operand rows allow 4-element vector loads
    int out_bf16, accumulate, relu;
    const float *bias;
    const char *mask; int64_t ldm; int mask_bf16;
    int gx, gy, S;                  // tiles along N, along M, reduction splits
    int c_staged;                   // bf16 kernel: write C through LDS in 16-byte pieces (no accumulate / split / row scale)
    const float *rscale;            // C[i,:] *= rscale[i] after everything else (fp32 C), or null
    // two products into one result, C = A W + A2 W2 (gemm_split_kernel<..., DUAL>): the reduction index runs over A's K1
    // columns, padded to K1p (whole steps), and then over A2's K - K1p columns; the cut weights lie one after the other
    const char *A2; int64_t lda2;
    int64_t K1, K1p;
};

// Tile of a workgroup in the one-dimensional grid.  Workgroup b runs on L2 domain b % NUM_XCD; the order is
// chosen so that workgroups that read the same operand data share a domain and follow one another there: the
// tiles of one reduction split (they read the same slab of both operands), or the tiles along N of one row
// block (they read the same rows of A).  Returns false for the padding workgroups at the end of the grid.
__device__ __forceinline__ bool tile_coords(const GemmArgs &g, int64_t b, int *bx, int *by, int *bz) {
    const int xcd = static_cast<int>(b % NUM_XCD);
    const int64_t seq = b / NUM_XCD;
    if (g.S > 1) {
        const int64_t tiles = static_cast<int64_t>(g.gx) * g.gy;
        const int64_t z = (seq / tiles) * NUM_XCD + xcd;
        const int64_t t = seq % tiles;
        *bz = static_cast<int>(z); *bx = static_cast<int>(t % g.gx); *by = static_cast<int>(t / g.gx);
        return z < g.S;
    }
    *bz = 0;
    *bx = static_cast<int>(seq % g.gx);
    const int64_t y = (seq / g.gx) * NUM_XCD + xcd;
    *by = static_cast<int>(y);
    return y < g.gy;
}
__device__ __forceinline__ bool tile_coords(const GemmArgs &g, int *bx, int *by, int *bz) { return tile_coords(g, blockIdx.x, bx, by, bz); }

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// four consecutive elements starting at element index `off` of a row; only the first nvalid are read
template <bool BF16>
__device__ __forceinline__ float4 load4(const char *base, int64_t off, int nvalid, int vec) {
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (nvalid <= 0) return r;
    if constexpr (BF16) {
        const uint16_t *p = reinterpret_cast<const uint16_t *>(base) + off;
        if (vec && nvalid >= 4) {
            uint2 v = *reinterpret_cast<const uint2 *>(p);
            r.x = __uint_as_float(v.x << 16); r.y = __uint_as_float(v.x & 0xffff0000u);
            r.z = __uint_as_float(v.y << 16); r.w = __uint_as_float(v.y & 0xffff0000u);
        } else {
            r.x = __uint_as_float(static_cast<uint32_t>(p[0]) << 16);
            if (nvalid > 1) r.y = __uint_as_float(static_cast<uint32_t>(p[1]) << 16);
            if (nvalid > 2) r.z = __uint_as_float(static_cast<uint32_t>(p[2]) << 16);
            if (nvalid > 3) r.w = __uint_as_float(static_cast<uint32_t>(p[3]) << 16);
        }
    } else {
        const float *p = reinterpret_cast<const float *>(base) + off;
        if (vec && nvalid >= 4) {
            r = *reinterpret_cast<const float4 *>(p);
        } else {
            r.x = p[0];
            if (nvalid > 1) r.y = p[1];
            if (nvalid > 2) r.z = p[2];
            if (nvalid > 3) r.w = p[3];
        }
    }
    return r;
}

__device__ __forceinline__ float epilogue_load(const char *p, int64_t at, int bf16) {
    return bf16 ? __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t *>(p)[at]) << 16) : reinterpret_cast<const float *>(p)[at];
}

// an element of the product with the whole epilogue (the sum with C included), as it is stored
__device__ __forceinline__ float epilogue_value(const GemmArgs &g, int64_t row, int64_t col, float v) {
    if (g.accumulate) v += epilogue_load(g.C, row * g.ldc + col, g.out_bf16);
    if (g.bias) v += g.bias[col];
    if (g.relu) v = v > 0.f ? v : 0.f;
    if (g.mask && !(epilogue_load(g.mask, row * g.ldm + col, g.mask_bf16) > 0.f)) v = 0.f;
    if (g.rscale) v *= g.rscale[row];
    return v;
}

// Writes one wave's TM x TN grid of 32x32 accumulator tiles (top-left corner (row0, col0)) with the epilogue.
// D layout of the 32x32 MFMAs: register r of lane l holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
template <int TM, int TN>
__device__ __forceinline__ void store_tile(const GemmArgs &g, const floatx16 (&acc)[TM][TN], int64_t row0, int64_t col0,
                                           int l32, int half, int bz) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t col = col0 + j * 32 + l32;
            if (col >= g.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = row0 + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                if (row >= g.M) continue;
                float v = acc[i][j][r];
                if (g.part) {
                    g.part[(static_cast<int64_t>(bz) * g.M + row) * g.N + col] = v;
                    continue;
                }
                v = epilogue_value(g, row, col, v);
                if (g.out_bf16) reinterpret_cast<uint16_t *>(g.C)[row * g.ldc + col] = static_cast<uint16_t>(f32_to_bf16_rne(v));
                else reinterpret_cast<float *>(g.C)[row * g.ldc + col] = v;
            }
        }
}

// The same through LDS: a wave rounds 32 rows of its accumulators at a time into a private LDS area (lds, STAGE_BYTES
// per wave) and leaves along the rows of C, 16 bytes per lane, so that a store instruction covers 4 rows x 256 bytes
// instead of 2 x 128 and the read-modify-write of an accumulating product moves whole vectors.  fp32 results only.
template <int TN> constexpr int STAGE_PITCH_T = TN * 32 + 8;  // floats per staged row (four rows further = other half of the banks)
template <int TN> constexpr int STAGE_BYTES_T = 32 * STAGE_PITCH_T<TN> * 4;   // per wave
constexpr int STAGE_BYTES = STAGE_BYTES_T<2>;

// TN: 32-column accumulator tiles side by side in the wave's part (2 or 1)
template <int TN>
__device__ __forceinline__ void store_tile_staged(const GemmArgs &g, const floatx16 (&acc)[2][TN], float *lds, int64_t row0,
                                                  int64_t col0, int lane, int bz) {
    constexpr int STAGE_PITCH = STAGE_PITCH_T<TN>;
    constexpr int CGS = TN * 8;                              // groups of four columns in a row
    constexpr int RPP = 64 / CGS;                            // rows per pass of the wave
    const int l32 = lane & 31, half = lane >> 5;
    float *dst = g.part ? g.part + static_cast<int64_t>(bz) * g.M * g.N : reinterpret_cast<float *>(g.C);
    const int64_t ld = g.part ? g.N : g.ldc;
    const bool vec = (reinterpret_cast<uintptr_t>(dst) % 16 == 0) && (ld % 4 == 0);
    const bool plain = g.part != nullptr;                   // partials take no epilogue
    const int cg = lane % CGS, rq = lane / CGS;             // the lane's column group (4 columns) and row within a pass
    const int64_t col = col0 + 4 * cg;
    float bv[4] = {0.f, 0.f, 0.f, 0.f};
    if (!plain && g.bias)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (col + e < g.N) bv[e] = g.bias[col + e];
    // what the epilogue reads of C, the mask and the row scales, before the first store, behind which it would wait; whole vectors from
    // clamped places (a wave's part of 32 columns: twice that takes the registers that the kernel's other waves need)
    constexpr bool EARLY = TN == 1;
    constexpr int NT_ = 32 / RPP;
    const bool whole = vec && col + 4 <= g.N;
    const bool mvec = g.mask && reinterpret_cast<uintptr_t>(g.mask) % 16 == 0 && g.ldm % 4 == 0;      // uniform over the grid
    auto clamped = [&](int i, int t) { const int64_t row = row0 + i * 32 + RPP * t + rq; return row < g.M ? row : g.M - 1; };
    const int64_t vcol = col + 4 <= g.N ? col : 0;      // (columns 0 .. 3: there where any vector is whole)
    float4 mk[2][NT_], ck[2][NT_];
    float rs[2][NT_];
    if (EARLY && !plain && mvec && g.N >= 4)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT_; ++t)
                mk[i][t] = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(g.mask) + clamped(i, t) * g.ldm + vcol);
    if (EARLY && !plain && g.accumulate && vec && g.N >= 4)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT_; ++t) ck[i][t] = *reinterpret_cast<const float4 *>(dst + clamped(i, t) * ld + vcol);
    if (EARLY && !plain && g.rscale)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < NT_; ++t) rs[i][t] = g.rscale[clamped(i, t)];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) lds[(8 * (r >> 2) + 4 * half + (r & 3)) * STAGE_PITCH + j * 32 + l32] = acc[i][j][r];
        __builtin_amdgcn_wave_barrier();
        if (col < g.N) {
#pragma unroll
            for (int t = 0; t < NT_; ++t) {
                const int lr = RPP * t + rq;
                const int64_t row = row0 + i * 32 + lr;
                if (row >= g.M) continue;
                const float4 v4 = *reinterpret_cast<const float4 *>(&lds[lr * STAGE_PITCH + 4 * cg]);
                float v[4] = {v4.x, v4.y, v4.z, v4.w};
                float *out = dst + row * ld + col;
                if (!plain) {
                    if (g.accumulate) {
                        if (whole) {
                            if (!EARLY) ck[i][t] = *reinterpret_cast<const float4 *>(out);
                            v[0] += ck[i][t].x; v[1] += ck[i][t].y; v[2] += ck[i][t].z; v[3] += ck[i][t].w;
                        } else {
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (col + e < g.N) v[e] += out[e];
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] += bv[e];
                        if (g.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
                    }
                    if (g.mask) {
                        if (mvec && col + 4 <= g.N) {
                            if (!EARLY) mk[i][t] = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(g.mask) + row * g.ldm + col);
                            const float m[4] = {mk[i][t].x, mk[i][t].y, mk[i][t].z, mk[i][t].w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] = m[e] > 0.f ? v[e] : 0.f;
                        } else {
                            const float *me = reinterpret_cast<const float *>(g.mask) + row * g.ldm + col;
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                if (col + e < g.N && !(me[e] > 0.f)) v[e] = 0.f;
                        }
                    }
                    if (g.rscale) {
                        if (!EARLY) rs[i][t] = g.rscale[row];
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] *= rs[i][t];
                    }
                }
                if (whole) {
                    *reinterpret_cast<float4 *>(out) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < g.N) out[e] = v[e];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

constexpr int BK = 16;
constexpr int PAD = 4;

// Stages one operand tile.  KC: the operand is stored with the reduction index contiguous
// (rows = output index); otherwise the output index is contiguous (rows = reduction index).
template <bool BF16, bool KC, int BT>
struct TileLoader {
    static constexpr int NLD = BT * BK / 4 / 256;   // float4 per thread
    float4 r[NLD];

    __device__ __forceinline__ void fetch(const char *base, int64_t ld, int64_t t0, int64_t T, int64_t k0,
                                          int64_t k_end, int vec, int tid) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q;
            if constexpr (KC) {
                const int row = idx >> 2, kq = idx & 3;
                const int64_t t = t0 + row, k = k0 + 4 * kq;
                const int nv = (t < T) ? static_cast<int>(k_end - k < 4 ? k_end - k : 4) : 0;
                r[q] = load4<BF16>(base, t * ld + k, nv, vec);
            } else {
                constexpr int QPR = BT / 4;
                const int kk = idx / QPR, tq = idx % QPR;
                const int64_t k = k0 + kk, t = t0 + 4 * tq;
                const int nv = (k < k_end) ? static_cast<int>(T - t < 4 ? T - t : 4) : 0;
                r[q] = load4<BF16>(base, k * ld + t, nv, vec);
            }
        }
    }

    // Interior tiles (every row of the tile exists, vector loads allowed) skip all range checks: the address of
    // each of the thread's vectors is formed once and then only stepped along the reduction index.
    const char *pf[NLD];

    __device__ __forceinline__ void fast_begin(const char *base, int64_t ld, int64_t t0, int64_t k0, int tid) {
        constexpr int ES = BF16 ? 2 : 4;
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q;
            if constexpr (KC) pf[q] = base + ((t0 + (idx >> 2)) * ld + k0 + 4 * (idx & 3)) * ES;
            else pf[q] = base + ((k0 + idx / (BT / 4)) * ld + t0 + 4 * (idx % (BT / 4))) * ES;
        }
    }

    __device__ __forceinline__ void fetch_fast(int64_t ld) {
        constexpr int ES = BF16 ? 2 : 4;
        const int64_t step = KC ? static_cast<int64_t>(BK) * ES : static_cast<int64_t>(BK) * ld * ES;
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            if constexpr (BF16) {
                const uint2 v = *reinterpret_cast<const uint2 *>(pf[q]);
                r[q] = make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                                   __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
            } else {
                r[q] = *reinterpret_cast<const float4 *>(pf[q]);
            }
            pf[q] += step;
        }
    }

    __device__ __forceinline__ void stash(float (*s)[BT + PAD], int tid) const {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q;
            if constexpr (KC) {
                const int row = idx >> 2, kq = idx & 3;
                s[4 * kq + 0][row] = r[q].x;
                s[4 * kq + 1][row] = r[q].y;
                s[4 * kq + 2][row] = r[q].z;
                s[4 * kq + 3][row] = r[q].w;
            } else {
                constexpr int QPR = BT / 4;
                const int kk = idx / QPR, tq = idx % QPR;
                *reinterpret_cast<float4 *>(&s[kk][4 * tq]) = r[q];
            }
        }
    }
};

template <bool BF16, bool A_KC, bool B_KC, int BM, int BN>
__global__ __launch_bounds__(256) void gemm_kernel(GemmArgs g) {
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int TM = WM / 32, TN = WN / 32;
    // operand tiles; fp32 results of full-size tiles leave through the same memory (store_tile_staged)
    constexpr int OPERAND_FLOATS = 2 * BK * (BM + PAD) + 2 * BK * (BN + PAD);
    constexpr bool STAGED = !BF16 && TM == 2 && TN == 2;
    constexpr int SMEM_FLOATS = (STAGED && 4 * STAGE_BYTES / 4 > OPERAND_FLOATS) ? 4 * STAGE_BYTES / 4 : OPERAND_FLOATS;
    __shared__ __attribute__((aligned(16))) float smem[SMEM_FLOATS];
    float (*As)[BK][BM + PAD] = reinterpret_cast<float (*)[BK][BM + PAD]>(smem);
    float (*Bs)[BK][BN + PAD] = reinterpret_cast<float (*)[BK][BN + PAD]>(smem + 2 * BK * (BM + PAD));

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (!tile_coords(g, &bx, &by, &bz)) return;      // uniform over the workgroup
    const int64_t m0 = static_cast<int64_t>(by) * BM;
    const int64_t n0 = static_cast<int64_t>(bx) * BN;
    const int64_t k_begin = static_cast<int64_t>(bz) * g.k_chunk;
    const int64_t k_end = (k_begin + g.k_chunk < g.K) ? k_begin + g.k_chunk : g.K;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    TileLoader<BF16, A_KC, BM> la;
    TileLoader<BF16, B_KC, BN> lb;
    const int64_t nk = (k_end > k_begin) ? (k_end - k_begin + BK - 1) / BK : 0;
    // uniform over the workgroup: the tile lies inside the matrices and both operands allow vector loads (measured
    // to pay only when the first operand is stored along the reduction index; X^T G keeps the checked loads)
    const bool interior = A_KC && m0 + BM <= g.M && n0 + BN <= g.N && g.a_vec && g.b_vec;
    const int64_t nk_full = (k_end > k_begin) ? (k_end - k_begin) / BK : 0;     // steps that need no check along k either
    if (nk > 0) {
        la.fetch(g.A, g.lda, m0, g.M, k_begin, k_end, g.a_vec, tid);
        lb.fetch(g.B, g.ldb, n0, g.N, k_begin, k_end, g.b_vec, tid);
        la.stash(As[0], tid);
        lb.stash(Bs[0], tid);
    }
    if (interior) {
        la.fast_begin(g.A, g.lda, m0, k_begin + BK, tid);
        lb.fast_begin(g.B, g.ldb, n0, k_begin + BK, tid);
    }
    // column sums of B (see gemm_small_kernel): a thread's vectors of a step cover the same four columns
    constexpr bool SUMS = !A_KC && !B_KC;
    const bool sums = SUMS && g.colpart && by == 0;
    double bsum[4] = {0.0, 0.0, 0.0, 0.0};
    auto add_b = [&]() __attribute__((always_inline)) {
        float t[4] = {lb.r[0].x, lb.r[0].y, lb.r[0].z, lb.r[0].w};
#pragma unroll
        for (int q = 1; q < TileLoader<BF16, B_KC, BN>::NLD; ++q) { t[0] += lb.r[q].x; t[1] += lb.r[q].y; t[2] += lb.r[q].z; t[3] += lb.r[q].w; }
#pragma unroll
        for (int e = 0; e < 4; ++e) bsum[e] += static_cast<double>(t[e]);
    };
    if (sums && nk > 0) add_b();
    __syncthreads();
    for (int64_t kt = 0; kt < nk; ++kt) {
        const int buf = static_cast<int>(kt & 1);
        const bool more = kt + 1 < nk;
        if (more) {
            if (interior && kt + 1 < nk_full) {
                la.fetch_fast(g.lda);
                lb.fetch_fast(g.ldb);
            } else {
                la.fetch(g.A, g.lda, m0, g.M, k_begin + (kt + 1) * BK, k_end, g.a_vec, tid);
                lb.fetch(g.B, g.ldb, n0, g.N, k_begin + (kt + 1) * BK, k_end, g.b_vec, tid);
            }
        }
        // operands of step kk+2 are read from LDS before the products of step kk are issued
        float a[2][TM], b[2][TN];
#pragma unroll
        for (int i = 0; i < TM; ++i) a[0][i] = As[buf][half][wm * WM + i * 32 + l32];
#pragma unroll
        for (int j = 0; j < TN; ++j) b[0][j] = Bs[buf][half][wn * WN + j * 32 + l32];
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 2) {
            const int cur = (kk >> 1) & 1;
            if (kk + 2 < BK) {
#pragma unroll
                for (int i = 0; i < TM; ++i) a[cur ^ 1][i] = As[buf][kk + 2 + half][wm * WM + i * 32 + l32];
#pragma unroll
                for (int j = 0; j < TN; ++j) b[cur ^ 1][j] = Bs[buf][kk + 2 + half][wn * WN + j * 32 + l32];
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][i], b[cur][j], acc[i][j], 0, 0, 0);
            // keep that order in the schedule: LDS reads of the next step, then this step's matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, TM * TN, 0);
        }
        if (more) {
            if (sums) add_b();
            la.stash(As[buf ^ 1], tid);
            lb.stash(Bs[buf ^ 1], tid);
        }
        __syncthreads();
    }

    if constexpr (SUMS) {
        if (sums) {     // the operand tiles are free: [256 / (BN / 4)][BN] partial sums
            double (*bred)[BN] = reinterpret_cast<double (*)[BN]>(smem);
            constexpr int QPR = BN / 4, ROWS = 256 / QPR;
            static_assert(ROWS * BN * sizeof(double) <= sizeof(smem), "the partial sums must fit the operand tiles");
#pragma unroll
            for (int e = 0; e < 4; ++e) bred[tid / QPR][4 * (tid % QPR) + e] = bsum[e];
            __syncthreads();
            if (tid < BN && n0 + tid < g.N) {
                double t = 0.0;
                for (int y = 0; y < ROWS; ++y) t += bred[y][tid];
                g.colpart[bz * g.N + n0 + tid] = static_cast<float>(t);
            }
            __syncthreads();
        }
    }
    if constexpr (STAGED) {
        // the last pass through the loop ended with a barrier: every wave is done with the operands
        store_tile_staged(g, acc, smem + wave * (STAGE_BYTES / 4), m0 + wm * WM, n0 + wn * WN, lane, bz);
    } else {
        store_tile<TM, TN>(g, acc, m0 + wm * WM, n0 + wn * WN, l32, half, bz);
    }
}

// ---------------------------------------------------------------------------------------------------
// bf16 operands on the bf16 matrix cores (v_mfma_f32_32x32x16_bf16: lane l supplies A[i = l%32][k = 8*(l/32) ..+7]
// and B[k = 8*(l/32) ..+7][j = l%32], eight consecutive k per lane).  Both operand tiles are kept in LDS with
// the reduction index contiguous (S[row][k], 32 k per step = four 16-byte chunks, rows padded to 80 bytes; the
// chunk position is XOR-ed with bits of the row so that neither the operand reads nor the transposing stores pile
// up on a few banks).  An operand stored with the reduction index contiguous is moved with 16-byte loads and
// stores.  One stored the other way is loaded 16 bytes along
// its rows, four consecutive k per thread, transposed in registers (byte permutes pair up the values of two k)
// and stored as 8-byte pieces: no 2-byte LDS traffic.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two fp32 numbers rounded to bf16 (nearest even), the first in the low half: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t bf16_pair(float x0, float x1) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{x0, x1}), bf16x2));
}
constexpr int HBK = 32;            // k per step of the bf16 kernel
constexpr int HPAD = 8;            // bf16 elements of row padding

// position (in elements) of 16-byte chunk `chunk` (0..3) inside LDS row `row`
__device__ __forceinline__ int chunk_pos(int row, int chunk) { return 8 * (chunk ^ ((row >> 3) & 3)); }

template <bool KC, int BT>
struct HalfTileLoader {
    static constexpr int NLD = KC ? BT * HBK / 8 / 256 : 4;   // 16-byte chunks per thread
    static constexpr int NTH = (HBK / 4) * (BT / 8);          // threads of the transposing path
    uint4 r[NLD];

    // eight consecutive bf16 starting at element `off`; only the first nvalid are read
    static __device__ __forceinline__ uint4 load8(const char *base, int64_t off, int nvalid) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (nvalid <= 0) return v;
        const uint16_t *p = reinterpret_cast<const uint16_t *>(base) + off;
        if (nvalid >= 8) return *reinterpret_cast<const uint4 *>(p);
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        for (int e = 0; e < nvalid; ++e) w[e >> 1] |= static_cast<uint32_t>(p[e]) << (16 * (e & 1));
        return make_uint4(w[0], w[1], w[2], w[3]);
    }

    int64_t k_rows = 0;             // rows of the operand when it is stored across the reduction index (set by the kernel)

    __device__ __forceinline__ void fetch(const char *base, int64_t ld, int64_t t0, int64_t T, int64_t k0, int64_t k_end,
                                          int tid) {
        if constexpr (KC) {
#pragma unroll
            for (int q = 0; q < NLD; ++q) {
                const int idx = tid + 256 * q;
                const int row = idx >> 2, kq = idx & 3;
                const int64_t t = t0 + row, k = k0 + 8 * kq;
                const int nv = (t < T) ? static_cast<int>(k_end - k < 8 ? k_end - k : 8) : 0;
                r[q] = load8(base, t * ld + k, nv);
            }
        } else {
            const int tt = tid;
            if (tt >= NTH) return;
            constexpr int CPR = BT / 8;
            const int kb = tt / CPR, tq = tt % CPR;       // four k starting at 4*kb, eight columns starting at 8*tq
            const int64_t t = t0 + 8 * tq;
            // a ragged last group of columns is still one 16-byte load where the row pitch covers it (every row but the
            // operand's last, whose padding need not exist): what the padding holds lands in result rows / columns beyond
            // the matrix, which are never stored
            const int exact = t >= T ? 0 : static_cast<int>(T - t < 8 ? T - t : 8);
            const int padded = (exact > 0 && t + 8 <= ld) ? 8 : exact;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int64_t k = k0 + 4 * kb + j;
                r[j] = load8(base, k * ld + t, k < k_end ? (k + 1 < k_rows ? padded : exact) : 0);
            }
        }
    }

    // check-free loads of interior tiles (operand stored along the reduction index): addresses formed once
    const char *pf[NLD];

    __device__ __forceinline__ void fast_begin(const char *base, int64_t ld, int64_t t0, int64_t k0, int tid) {
        static_assert(KC, "the check-free path serves operands stored along the reduction index");
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + 256 * q;
            pf[q] = base + ((t0 + (idx >> 2)) * ld + k0 + 8 * (idx & 3)) * 2;
        }
    }

    __device__ __forceinline__ void fetch_fast() {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            r[q] = *reinterpret_cast<const uint4 *>(pf[q]);
            pf[q] += HBK * 2;
        }
    }

    __device__ __forceinline__ void stash(uint16_t (*s)[HBK + HPAD], int tid) const {
        if constexpr (KC) {
#pragma unroll
            for (int q = 0; q < NLD; ++q) {
                const int idx = tid + 256 * q;
                const int row = idx >> 2, kq = idx & 3;
                *reinterpret_cast<uint4 *>(&s[row][chunk_pos(row, kq)]) = r[q];
            }
        } else {
            const int tt = tid;
            if (tt >= NTH) return;
            constexpr int CPR = BT / 8;
            const int kb = tt / CPR, tq = tt % CPR;
            const uint32_t w[4][4] = {{r[0].x, r[0].y, r[0].z, r[0].w}, {r[1].x, r[1].y, r[1].z, r[1].w},
                                      {r[2].x, r[2].y, r[2].z, r[2].w}, {r[3].x, r[3].y, r[3].z, r[3].w}};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                // column 8*tq+e of the four k: the low (e even) or high (e odd) halves of word e/2 of the four rows
                const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                uint2 v;
                v.x = __builtin_amdgcn_perm(w[1][e >> 1], w[0][e >> 1], sel);
                v.y = __builtin_amdgcn_perm(w[3][e >> 1], w[2][e >> 1], sel);
                const int row = 8 * tq + e;
                *reinterpret_cast<uint2 *>(&s[row][chunk_pos(row, kb >> 1) + 4 * (kb & 1)]) = v;
            }
        }
    }
};

__device__ __forceinline__ bool positive_bf16(uint32_t bits) { return __uint_as_float(bits << 16) > 0.f; }

// eight bf16: those of v where m > 0, else zero
__device__ __forceinline__ uint4 keep_positive(uint4 v, uint4 m) {
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
    const uint32_t k[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
    for (int d = 0; d < 4; ++d)
        w[d] &= (positive_bf16(k[d] & 0xffffu) ? 0xffffu : 0u) | (__uint_as_float(k[d] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// (X^T G, both of whose operands are stored across the reduction index, has gemm_bf16_cols_kernel)
template <bool A_KC, bool B_KC, int BM, int BN>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmArgs g) {
    constexpr int WM = BM / 2, WN = BN / 2;
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int LDSROW = HBK + HPAD;
    constexpr int CPITCH = BN + 8;          // row pitch of the staged output tile (16-byte multiple)
    static_assert(BM * CPITCH <= 2 * (BM + BN) * LDSROW, "the staged output tile must fit the operand buffers");
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 * (BM + BN) * LDSROW];
    uint16_t (*As)[BM][LDSROW] = reinterpret_cast<uint16_t (*)[BM][LDSROW]>(smem);
    uint16_t (*Bs)[BN][LDSROW] = reinterpret_cast<uint16_t (*)[BN][LDSROW]>(smem + 2 * BM * LDSROW);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (!tile_coords(g, &bx, &by, &bz)) return;      // uniform over the workgroup
    const int64_t m0 = static_cast<int64_t>(by) * BM;
    const int64_t n0 = static_cast<int64_t>(bx) * BN;
    const int64_t k_begin = static_cast<int64_t>(bz) * g.k_chunk;
    const int64_t k_end = (k_begin + g.k_chunk < g.K) ? k_begin + g.k_chunk : g.K;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    HalfTileLoader<A_KC, BM> la;
    HalfTileLoader<B_KC, BN> lb;
    la.k_rows = g.K; lb.k_rows = g.K;
    const int64_t nk = (k_end > k_begin) ? (k_end - k_begin + HBK - 1) / HBK : 0;
    if (nk > 0) {
        la.fetch(g.A, g.lda, m0, g.M, k_begin, k_end, tid);
        lb.fetch(g.B, g.ldb, n0, g.N, k_begin, k_end, tid);
        la.stash(As[0], tid);
        lb.stash(Bs[0], tid);
    }
    // uniform over the workgroup: both operands are stored along the reduction index and the tile lies inside
    constexpr bool FAST = A_KC && B_KC;
    const bool interior = FAST && m0 + BM <= g.M && n0 + BN <= g.N;
    const int64_t nk_full = (k_end > k_begin) ? (k_end - k_begin) / HBK : 0;
    if constexpr (FAST) {
        if (interior) {
            la.fast_begin(g.A, g.lda, m0, k_begin + HBK, tid);
            lb.fast_begin(g.B, g.ldb, n0, k_begin + HBK, tid);
        }
    }
    __syncthreads();
    for (int64_t kt = 0; kt < nk; ++kt) {
        const int buf = static_cast<int>(kt & 1);
        const bool more = kt + 1 < nk;
        if (more) {
            bool done = false;
            if constexpr (FAST) {
                if (interior && kt + 1 < nk_full) {
                    la.fetch_fast();
                    lb.fetch_fast();
                    done = true;
                }
            }
            if (!done) {
                la.fetch(g.A, g.lda, m0, g.M, k_begin + (kt + 1) * HBK, k_end, tid);
                lb.fetch(g.B, g.ldb, n0, g.N, k_begin + (kt + 1) * HBK, k_end, tid);
            }
        }
#pragma unroll
        for (int ks = 0; ks < HBK; ks += 16) {
            bf16x8 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * WM + i * 32 + l32;
                a[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&As[buf][row][chunk_pos(row, ks / 8 + half)]));
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row = wn * WN + j * 32 + l32;
                b[j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(&Bs[buf][row][chunk_pos(row, ks / 8 + half)]));
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (more) {
            la.stash(As[buf ^ 1], tid);
            lb.stash(Bs[buf ^ 1], tid);
        }
        __syncthreads();
    }
    if (!g.c_staged) {
        store_tile<TM, TN>(g, acc, m0 + wm * WM, n0 + wn * WN, l32, half, bz);
        return;
    }
    // bf16 output without a read-modify-write epilogue: the tile is rounded into LDS (the operand buffers are free
    // after the last barrier) and leaves in 16-byte pieces along the rows, instead of 2 bytes per lane.
    uint16_t (*Cs)[CPITCH] = reinterpret_cast<uint16_t (*)[CPITCH]>(smem);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int col = wn * WN + j * 32 + l32;
            const float bv = (g.bias && n0 + col < g.N) ? g.bias[n0 + col] : 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm * WM + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                float v = acc[i][j][r] + bv;
                if (g.relu) v = v > 0.f ? v : 0.f;
                Cs[row][col] = static_cast<uint16_t>(f32_to_bf16_rne(v));
            }
        }
    __syncthreads();
    constexpr int CQ = BN / 8;
    for (int c = tid; c < BM * CQ; c += 256) {
        const int row = c / CQ, cq = c % CQ;
        const int64_t grow = m0 + row, gcol = n0 + 8 * cq;
        if (grow >= g.M || gcol >= g.N) continue;
        uint16_t *dst = reinterpret_cast<uint16_t *>(g.C) + grow * g.ldc + gcol;
        uint4 v = *reinterpret_cast<const uint4 *>(&Cs[row][8 * cq]);
        if (gcol + 8 <= g.N) {
            if (g.mask) v = keep_positive(v, *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(g.mask) + grow * g.ldm + gcol));
            *reinterpret_cast<uint4 *>(dst) = v;
        } else {
            for (int e = 0; gcol + e < g.N; ++e)
                dst[e] = g.mask && !positive_bf16(reinterpret_cast<const uint16_t *>(g.mask)[grow * g.ldm + gcol + e]) ? 0 : Cs[row][8 * cq + e];
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// bf16 products of many rows with a small weight matrix (C = A W or A W^T, at most 512 k, more than 64 columns), which move far
// more bytes than they compute: memory bounds them.  A workgroup of NS waves walks tiles of 32 rows and all its life holds its
// columns of W in registers, 32 per wave, in the layout the matrix instruction reads (KS units of 16 k): a tile costs its rows of A
// and of C and nothing else, A is read once per 256 columns, and all of a tile's loads go out at once, two tiles ahead.  One barrier
// per tile: rows of A and rounded results have two LDS buffers each.  Loads and stores of a wave complete in order, so every tile
// issues the same ones, unconditionally (the last row's tile comes apart, at the end; stores beyond the matrix go to an offset that
// the buffer's bounds drop): nothing waits for a store.  Results are stored past the caches (they are read once, by a later
// kernel, and mostly larger than what the caches hold): 980 k x 256 x 128 153 -> 125 us, 980 k x 256 x 47 124 -> 99.
// The operands of the instruction are exchanged (W first): a lane then holds four neighbouring columns of a row of C.
// us, gemm_bf16_kernel's tiles of 128 columns -> here, TB/s of operand and result: 980 k x 256 x 256 322 -> 195 (5.1), x 128 231 ->
// 123 (6.1), x 47 261 -> 96 (6.2), 150 k x 256 x 512 82 -> 50 (4.6), 200 k x 128 x 128 36 -> 21 (5.0).
constexpr int stream_lds(int KS, int NS) { return 2 * (2 * KS * 34 * 16) + 2 * (32 * (NS * 32 + 8) * 2) + NS * 128; }
// workgroups per compute unit: what its LDS holds, and at most 16 waves with their weights
constexpr int stream_held(int KS, int NS) { return std::min(160 * 1024 / stream_lds(KS, NS), std::max(1, (KS == 32 ? 8 : 16) / NS)); }

template <int KS, int NS, bool MASK>
__global__ __launch_bounds__(NS * 64, std::max(1, stream_held(KS, NS) * NS / 4)) void gemm_bf16_stream_kernel(GemmArgs g, const uint16_t *Wt, uint32_t n_pad) {
    constexpr int NT = NS * 64, NU = 2 * KS, PLANE = 34, A_BYTES = NU * PLANE * 16;     // 16-byte units (k / 8, row), see Units16
    constexpr int NLD = 32 * NU / NT, RPP = NT / NU;                                    // loads per thread and tile, rows per pass
    constexpr int CPITCH = NS * 32 + 8, C_BYTES = 32 * CPITCH * 2;
    static_assert(NT % NU == 0 && 32 * NU % NT == 0, "whole rows per pass");
    __shared__ __attribute__((aligned(16))) char smem[2 * A_BYTES + 2 * C_BYTES + NS * 128];
    static_assert(sizeof(smem) == stream_lds(KS, NS), "LDS of a workgroup");
    float *bias = reinterpret_cast<float *>(smem + 2 * A_BYTES + 2 * C_BYTES);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int n0 = static_cast<int>(blockIdx.y) * (NS * 32);
    const int64_t full = (g.M - 1) / 32;                // tiles before the one that holds the last row

    for (int c = tid; c < NS * 32; c += NT) bias[c] = (g.bias && n0 + c < g.N) ? g.bias[n0 + c] : 0.f;
    bf16x8 w[KS];       // (a wave beyond the last column of the image holds its last columns: never stored)
    {
        const uint32_t n = static_cast<uint32_t>(n0 + wave * 32) + 32 <= n_pad ? n0 + wave * 32 : n_pad - 32;
#pragma unroll
        for (int s = 0; s < KS; ++s)
            w[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Wt + (static_cast<size_t>(2 * s + half) * n_pad + n + l32) * 8));
    }
    const int v = tid % NU, r0 = tid / NU;              // the thread's vector of a row of A, its first row
    const int K = static_cast<int>(g.K), have = K - 8 * v;                    // elements of that vector that exist
    const uint32_t a_off = static_cast<uint32_t>(r0) * static_cast<uint32_t>(g.lda) * 2 +
                           16u * (have > 0 ? v : (K - 1) / 8);                // (vectors beyond the width read the last one and are cleared)
    const uint32_t a_step = static_cast<uint32_t>(g.lda) * 2 * RPP;
    typedef uint4 Rows[NLD];
    auto load = [&](int64_t t, Rows &r) __attribute__((always_inline)) {
        const char *base = g.A + (t < full ? t : full - 1) * 64 * g.lda;
#pragma unroll
        for (int q = 0; q < NLD; ++q) r[q] = *reinterpret_cast<const uint4 *>(base + (a_off + q * a_step));
    };
    auto load_last = [&](Rows &r) __attribute__((always_inline)) {            // the rows that exist, no further than their width
        const int rows = static_cast<int>(g.M - full * 32);
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int row = r0 + q * RPP;
            r[q] = HalfTileLoader<true, 128>::load8(g.A, (full * 32 + row) * g.lda + 8 * v, row < rows ? (have < 8 ? have : 8) : 0);
        }
    };
    auto put = [&](Rows &r, char *As) __attribute__((always_inline)) {
        if (K < KS * 16) {
#pragma unroll
            for (int q = 0; q < NLD; ++q) {
                uint32_t x[4] = {r[q].x, r[q].y, r[q].z, r[q].w};
#pragma unroll
                for (int d = 0; d < 4; ++d) x[d] = 2 * d + 1 < have ? x[d] : 2 * d < have ? x[d] & 0xffffu : 0u;
                r[q] = make_uint4(x[0], x[1], x[2], x[3]);
            }
        }
#pragma unroll
        for (int q = 0; q < NLD; ++q) *reinterpret_cast<uint4 *>(As + (v * PLANE + r0 + q * RPP) * 16) = r[q];
    };
    // the thread's two pieces of a finished tile: 8 columns of rows cr and cr + 16
    const int cr = tid / (NS * 4), cc = 8 * (tid % (NS * 4));
    const uint32_t ldc2 = static_cast<uint32_t>(g.ldc) * 2, ldm2 = static_cast<uint32_t>(g.ldm) * 2;
    const bool whole = n0 + cc + 8 <= g.N;
    const bool cut = !MASK && n0 + NS * 32 > g.N && g.N % 8 != 0;             // a group of eight columns ends inside the matrix (uniform; see bf16_stream_rows)

    // mid: what becomes of the A registers between the products and the barrier
    auto tile = [&](int64_t t, int rows, int buf, auto mid) __attribute__((always_inline)) {
        if constexpr (MASK) asm("" : "+s"(t));         // (addresses per tile: pointers carried from tile to tile take registers that the weights need)
        const char *As = smem + buf * A_BYTES;
        uint16_t *Cs = reinterpret_cast<uint16_t *>(smem + 2 * A_BYTES + buf * C_BYTES);
        const int64_t m0 = t * 32;
        uint4 mk[2];
        if constexpr (MASK) {
            const char *mbase = g.mask + m0 * g.ldm * 2;
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int row = cr + 16 * p < rows ? cr + 16 * p : rows - 1;
                mk[p] = *reinterpret_cast<const uint4 *>(mbase + (static_cast<uint32_t>(row) * ldm2 + (whole ? 2u * (n0 + cc) : 0u)));
            }
        }
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8 x = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(As + ((2 * s + half) * PLANE + l32) * 16));
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[s], x, acc, 0, 0, 0);
        }
        // four operand reads ahead of the matrix instructions
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int s = 0; s < KS - 4; ++s) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {                    // registers 4 q ..: columns 8 q + 4 half .. of row l32
            const float4 b4 = *reinterpret_cast<const float4 *>(&bias[wave * 32 + 8 * q + 4 * half]);
            float x[4] = {acc[4 * q] + b4.x, acc[4 * q + 1] + b4.y, acc[4 * q + 2] + b4.z, acc[4 * q + 3] + b4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = g.relu && !(x[e] > 0.f) ? 0.f : x[e];
            uint2 o;
            o.x = bf16_pair(x[0], x[1]);
            o.y = bf16_pair(x[2], x[3]);
            *reinterpret_cast<uint2 *>(&Cs[l32 * CPITCH + wave * 32 + 8 * q + 4 * half]) = o;
        }
        mid();
        __syncthreads();
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc(g.C + (m0 * g.ldc + n0) * 2, 0, 0x7fffffff, 0x00027000);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint4 o = *reinterpret_cast<const uint4 *>(&Cs[(cr + 16 * p) * CPITCH + cc]);
            if constexpr (MASK) o = keep_positive(o, mk[p]);
            const uint32_t at = cr + 16 * p < rows && whole ? (cr + 16 * p) * ldc2 + 2u * cc : 0xfffffff0u;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rsrc, at, 0, 2);
        }
        if (cut) {
#pragma unroll 1
            for (int e = 0; e < 16; ++e) {
                const int row = cr + 2 * (e & 8), col = cc + (e & 7);
                const bool in = !whole && row < rows && n0 + col < g.N;
                __builtin_amdgcn_raw_buffer_store_b16(Cs[row * CPITCH + col], rsrc, in ? row * ldc2 + 2u * col : 0xfffffff0u, 0, 0);
            }
        }
    };
    // as many dropped stores as the tiles before would have issued, so that the waits of the loop can allow for them
    auto dropped = [&](uint32_t at) __attribute__((always_inline)) {
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc(g.C, 0, 0x7fffffff, 0x00027000);
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, rsrc, at, 0, 2);
        __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, rsrc, at + 16, 0, 0);
    };
    Rows ra, rb;
    const int64_t step = gridDim.x;
    int64_t t = blockIdx.x;
    if (t < full) {                                      // uniform over the workgroup
        load(t, ra);
        load(t + step, rb);
        dropped(0xffffff00u);
        put(ra, smem);
        load(t + 2 * step, ra);
        dropped(0xffffff40u);
        __syncthreads();
        for (; t + step < full; t += 2 * step) {         // (one way out: the waits are counted over every path)
            tile(t, 32, 0, [&]() { put(rb, smem + A_BYTES); load(t + 3 * step, rb); });
            tile(t + step, 32, 1, [&]() { put(ra, smem); load(t + 4 * step, ra); });
        }
        if (t < full) {
            tile(t, 32, 0, []() {});
            t += step;
        }
        __syncthreads();                                 // both buffers of A are free
    }
    if (t == full) {                                     // the tile with the last row (t went through every residue: one workgroup's)
        load_last(ra);
        put(ra, smem);
        __syncthreads();
        tile(t, static_cast<int>(g.M - full * 32), 0, []() {});
    }
}

// ---------------------------------------------------------------------------------------------------
// fp32 operands on the bf16 matrix cores.  An fp32 number is the exact sum of three bf16 numbers (its 24 significant
// bits cut into 8 + 8 + 8, with signs), so a product a * b is the sum of nine bf16 products, each exact in fp32.  The
// three smallest (together at most 2^-23 of the product: the size of fp32's own rounding) are dropped, the other six
// are accumulated in fp32 by v_mfma_f32_32x32x16_bf16, smallest first.  Six such instructions cover the k-range of
// eight v_mfma_f32_32x32x2_f32 at about a fifteenth of the cost each.
//
// LDS holds the three pieces of both operand tiles, 32 k per step, in one buffer (the next step's operands wait in
// registers; two workgroups share a compute unit and fill one another's barriers).  An operand stored along the
// reduction index is cut while it is staged and kept in 16-byte units S[piece][k / 8][row] (a lane's eight k are one
// 16-byte read, consecutive lanes read consecutive units; a plane is 32 bytes longer than a power of two so that the
// 8-byte staging stores of 16 consecutive lanes, 2 rows x 4 units x 2 halves, cover 128 consecutive bytes of banks);
// the weight matrix of a plain product is cut once, by split_repack_kernel, into the same units in global memory and
// only copied here.  Both operands of X^T G are stored across the reduction index: gemm_split_cols_kernel reads
// them straight into registers instead.
constexpr int SBK = 32;

// x = piece 0 + piece 1 + piece 2 exactly, for two numbers at once; p[i] holds piece i of x0 in its low half and of
// x1 in its high half.  Rounding to nearest bounds the second piece by 2^-8 |x| and the third by 2^-16 |x|; the
// remainders are exact fp32 differences with at most 16 and 8 significant bits.
__device__ __forceinline__ void split3_pair(float x0, float x1, uint32_t (&p)[3]) {
    p[0] = bf16_pair(x0, x1);
    const float r0 = x0 - __uint_as_float(p[0] << 16), r1 = x1 - __uint_as_float(p[0] & 0xffff0000u);
    p[1] = bf16_pair(r0, r1);
    const float s0 = r0 - __uint_as_float(p[1] << 16), s1 = r1 - __uint_as_float(p[1] & 0xffff0000u);
    p[2] = bf16_pair(s0, s1);
}

// 16-byte units of an operand kept along the reduction index: unit (piece, u = k / 8, row)
template <int BT>
struct Units16 {
    static constexpr int PLANE = BT + 2;                    // units per (piece, u) plane
    static constexpr int BYTES = 3 * 4 * PLANE * 16;
    static __device__ __forceinline__ int at(int piece, int u, int row) { return ((piece * 4 + u) * PLANE + row) * 16; }
};

// operand stored along the reduction index, cut while staged: a row's 32 k are eight float4 of eight threads
template <int BT, int NT = 256>
struct SplitRowLoader {
    static constexpr int NLD = BT * SBK / 4 / NT;
    float4 r[NLD];
    const char *pf[NLD];

    __device__ __forceinline__ void fetch(const char *base, int64_t ld, int64_t t0, int64_t T, int64_t k0, int64_t k_end,
                                          int vec, int tid) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + NT * q;
            const int row = idx >> 3, kq = idx & 7;
            const int64_t t = t0 + row, k = k0 + 4 * kq;
            const int nv = (t < T) ? static_cast<int>(k_end - k < 4 ? k_end - k : 4) : 0;
            r[q] = load4<false>(base, t * ld + k, nv, vec);
        }
    }

    __device__ __forceinline__ void fast_begin(const char *base, int64_t ld, int64_t t0, int64_t k0, int tid) {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + NT * q;
            pf[q] = base + ((t0 + (idx >> 3)) * ld + k0 + 4 * (idx & 7)) * 4;
        }
    }

    __device__ __forceinline__ void fetch_fast() {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            r[q] = *reinterpret_cast<const float4 *>(pf[q]);
            pf[q] += SBK * 4;
        }
    }

    // check-free loads of one step at a given place (rows t0.., 32 k from k0): no state between steps.  The tile's
    // corner is uniform over the workgroup, a thread adds a 32-bit offset inside the tile (ld < 2^22 elements).
    __device__ __forceinline__ void fetch_at(const char *base, int64_t ld, int64_t t0, int64_t k0, int tid) {
        const char *corner = base + (t0 * ld + k0) * 4;
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + NT * q;
            const uint32_t off = (static_cast<uint32_t>(idx >> 3) * static_cast<uint32_t>(ld) + 4u * (idx & 7)) * 4u;
            r[q] = *reinterpret_cast<const float4 *>(corner + off);
        }
    }

    uint2 pk[NLD][3];               // the pieces of r, ready for LDS

    __device__ __forceinline__ void cut() {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            uint32_t lo[3], hi[3];
            split3_pair(r[q].x, r[q].y, lo);
            split3_pair(r[q].z, r[q].w, hi);
#pragma unroll
            for (int p = 0; p < 3; ++p) pk[q][p] = make_uint2(lo[p], hi[p]);
        }
    }

    __device__ __forceinline__ void put(char *s, int tid) const {
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int idx = tid + NT * q;
            const int row = idx >> 3, kq = idx & 7;
#pragma unroll
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<uint2 *>(s + Units16<BT>::at(p, kq >> 1, row) + 8 * (kq & 1)) = pk[q][p];
        }
    }
};

// second operand already cut into units Wt[piece][k / 8][n] (n padded to whole tiles, k to whole steps): plain copies

template <int BT, int NT = 256>
struct SplitPlaneLoader {
    static constexpr int NLD = 3 * 4 * BT / NT;
    u32x4 r[NLD];
    const u32x4 *pf;                // the thread's first unit; its others lie q * stride_q further on
    int64_t stride_q;               // in units

    // ku_total: 16-byte units along k of one piece; n_pad: rows of a plane.  NT consecutive units of the LDS image
    // (piece, u, row) are NT / BT planes of BT rows: thread tid copies row tid % BT of planes tid / BT + q * NT / BT.
    __device__ __forceinline__ void begin(const uint16_t *Wt, int64_t ku_total, int64_t n_pad, int64_t t0, int64_t k0, int tid) {
        static_assert((BT == 128 || BT == 64) && (NT / BT == 2 || NT / BT == 4), "planes per pass: 2 or 4, both divide the 4 units of a piece");
        const int pu = tid / BT, row = tid % BT;
        pf = reinterpret_cast<const u32x4 *>(Wt) + (k0 / 8 + pu) * n_pad + t0 + row;
        stride_q = (NT / BT) * n_pad;
        piece_stride = (ku_total - 4) * n_pad;
    }
    int64_t piece_stride;           // extra distance when q crosses into the next piece

    __device__ __forceinline__ void fetch(int64_t n_pad) {
        constexpr int PPQ = NT / BT;           // planes per pass
#pragma unroll
        for (int q = 0; q < NLD; ++q) r[q] = pf[q * stride_q + ((q * PPQ) / 4) * piece_stride];
        pf += (SBK / 8) * n_pad;
    }

    __device__ __forceinline__ void stash(char *s, int tid) const {
        constexpr int PPQ = NT / BT;
        const int pu0 = tid / BT, row = tid % BT;
#pragma unroll
        for (int q = 0; q < NLD; ++q) {
            const int pu = pu0 + q * PPQ;
            *reinterpret_cast<u32x4 *>(s + Units16<BT>::at(pu >> 2, pu & 3, row)) = r[q];
        }
    }
};

// C = A B (or A B^T) with A stored along the reduction index; the second operand comes cut into units (Wt: ku_total
// units along k per piece, n_pad rows).  NW waves: four (2 x 2) or, on a 128 x 128 tile, eight (2 x 4, each a 64 x 32
// part: half the staging and half the accumulators per thread, four waves per SIMD).
template <int BM, int BN, int NW = 4, bool DUAL = false>
__global__ __launch_bounds__(NW * 64, NW / 2) void gemm_split_kernel(GemmArgs g, const uint16_t *Wt, int64_t ku_total, int64_t n_pad) {
    static_assert(NW == 4 || (NW == 8 && BN == 128), "eight waves: 128 columns");
    constexpr int NT = NW * 64;
    constexpr int WM = BM / 2, WN = BN / (NW / 2);
    constexpr int TM = WM / 32, TN = WN / 32;
    constexpr int A_BYTES = Units16<BM>::BYTES;
    constexpr int B_BYTES = Units16<BN>::BYTES;
    __shared__ __attribute__((aligned(16))) char smem[A_BYTES + B_BYTES];
    char *As = smem, *Bs = smem + A_BYTES;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / (NW / 2), wn = wave % (NW / 2);
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (!tile_coords(g, &bx, &by, &bz)) return;      // uniform over the workgroup
    const int64_t m0 = static_cast<int64_t>(by) * BM;
    const int64_t n0 = static_cast<int64_t>(bx) * BN;
    const int64_t k_begin = static_cast<int64_t>(bz) * g.k_chunk;
    const int64_t k_end = (k_begin + g.k_chunk < g.K) ? k_begin + g.k_chunk : g.K;

    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    SplitRowLoader<BM, NT> la_r;
    SplitPlaneLoader<BN, NT> lb_p;
    const int64_t nk = (k_end > k_begin) ? (k_end - k_begin + SBK - 1) / SBK : 0;
    const int64_t nk_full = (k_end > k_begin) ? (k_end - k_begin) / SBK : 0;
    // uniform over the workgroup: every row of the tile exists and vector loads are allowed
    const bool interior = m0 + BM <= g.M && g.a_vec;
    if (nk > 0) {
        la_r.fetch(g.A, g.lda, m0, g.M, k_begin, DUAL ? g.K1 : k_end, g.a_vec, tid);      // DUAL: one split, k_begin = 0
        lb_p.begin(Wt, ku_total, n_pad, n0, k_begin, tid);
        lb_p.fetch(n_pad);
        la_r.cut();
        la_r.put(As, tid);
        lb_p.stash(Bs, tid);
        if (!DUAL && interior) la_r.fast_begin(g.A, g.lda, m0, k_begin + SBK, tid);
    }
    __syncthreads();
    // the products of one step (32 k) out of LDS; CUT: the first operand of the next step, which waits in registers, is
    // cut into its pieces between the matrix instructions of the second half (about five vector instructions fit
    // behind each matrix instruction's issue; measured: 4 %)
    auto products = [&](auto cut_tag) {
        constexpr bool CUT = decltype(cut_tag)::value;
#pragma unroll
        for (int ks = 0; ks < SBK / 16; ++ks) {
            // nothing of the second half moves into the first: the loads of the next operands get that long to arrive
            if (CUT && ks == SBK / 16 - 1) __builtin_amdgcn_sched_barrier(0);
            bf16x8 a[3][TM], b[3][TN];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int row = wm * WM + i * 32 + l32;
                    a[p][i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(As + Units16<BM>::at(p, 2 * ks + half, row)));
                }
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int row = wn * WN + j * 32 + l32;
                    b[p][j] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Bs + Units16<BN>::at(p, 2 * ks + half, row)));
                }
            }
            if (CUT && ks == SBK / 16 - 1) la_r.cut();
            // the six piece products, smallest first
#define CG_PIECES(PA_, PB_)                                                                                                  \
    _Pragma("unroll") for (int i = 0; i < TM; ++i) _Pragma("unroll") for (int j = 0; j < TN; ++j)                            \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[PA_][i], b[PB_][j], acc[i][j], 0, 0, 0);
            CG_PIECES(2, 0) CG_PIECES(0, 2) CG_PIECES(1, 1) CG_PIECES(1, 0) CG_PIECES(0, 1) CG_PIECES(0, 0)
#undef CG_PIECES
            if (CUT && ks == SBK / 16 - 1) {
#pragma unroll
                for (int t = 0; t < 6 * TM * TN; ++t) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one matrix instruction
                    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);      // vector instructions behind it
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    for (int64_t kt = 0; kt + 1 < nk; ++kt) {
        if constexpr (DUAL) {
            // which of the two first operands this step reads is uniform over the grid; the check-free loads form their
            // addresses from it (no per-thread pointers to carry across the change of operand)
            const int64_t k0 = (kt + 1) * SBK;
            const bool second = k0 >= g.K1p;
            const char *base = second ? g.A2 : g.A;
            const int64_t ld = second ? g.lda2 : g.lda;
            const int64_t kk = second ? k0 - g.K1p : k0, kend = second ? g.K - g.K1p : g.K1;
            if (interior && kk + SBK <= kend) la_r.fetch_at(base, ld, m0, kk, tid);
            else la_r.fetch(base, ld, m0, g.M, kk, kend, g.a_vec, tid);
        } else {
            if (interior && kt + 1 < nk_full) la_r.fetch_fast();
            else la_r.fetch(g.A, g.lda, m0, g.M, k_begin + (kt + 1) * SBK, k_end, g.a_vec, tid);
        }
        lb_p.fetch(n_pad);
        products(std::true_type{});
        __syncthreads();            // every wave has read this step's operands
        la_r.put(As, tid);
        lb_p.stash(Bs, tid);
        __syncthreads();
    }
    if (nk > 0) products(std::false_type{});
    if constexpr (TM == 2 && (TN == 2 || TN == 1)) {
        static_assert(NW * STAGE_BYTES_T<TN> <= A_BYTES + B_BYTES, "the staged output must fit the operand buffers");
        __syncthreads();                    // every wave is done with the operands
        store_tile_staged<TN>(g, acc, reinterpret_cast<float *>(smem + wave * STAGE_BYTES_T<TN>), m0 + wm * WM, n0 + wn * WN, lane, bz);
    } else {
        store_tile<TM, TN>(g, acc, m0 + wm * WM, n0 + wn * WN, l32, half, bz);
    }
}

// ---------------------------------------------------------------------------------------------------
// The same product for many rows and a small weight matrix (at most 256 columns and 256 k, the sum of two products among them), where
// a tile's life of a few steps leaves gemm_split_kernel waiting for its first operands and its last stores.  A workgroup walks tiles of
// 32 rows and all its life holds the three pieces of its weights in registers: a wave 32 columns and 128 k (96 registers, so that two
// waves share a SIMD; one wave per SIMD with 192 or 384 of them was no faster than gemm_split_kernel).  Above 128 k the waves halve the reduction between them (KH = 2), exchange half of their partial tiles through LDS and store
// half of the rows each.  Rows of A are fetched two tiles ahead and cut behind the matrix instructions (cut after them: 1-2 % slower);
// LDS holds A's pieces, one tile being stored while the other is multiplied: one barrier per tile.  Units of 16 bytes
// S[k / 128][piece][k / 8][row], a plane one unit longer than 32 rows: the units that 8 lanes store lie 4 banks apart.
// As in gemm_bf16_stream_kernel the operands are exchanged, every tile issues the same loads and stores unconditionally (those
// beyond the matrix are dropped by the buffer's bounds) and the last row's tile comes apart.
// us, in a 306 k-vertex GraphSAGE epoch, gemm_split_kernel -> here: sum of two products of 100 k 244 -> 205, masked sum of two of 47 k 206
// -> 126 (5.9 TB/s: memory), 256 x 256 246 -> 204 (1.2 PFLOP/s of bf16 work; a single product alone 265 -> 238, see split_stream_pays); error against fp64 2.4e-7 -> 1.7e-7 (shorter chains).
constexpr int split_stream_slots(int NS, int KH) { return KH == 1 ? NS : 2 * NS / KH; }     // 32 x 32 parts of C on their way through LDS
constexpr int split_stream_lds(int NS, int KH) { return 2 * KH * 3 * 16 * 33 * 16 + split_stream_slots(NS, KH) * 32 * 36 * 4 + NS / KH * 128; }
constexpr int split_stream_held(int NS, int KH) { return NS == 4 && KH == 1 ? 2 : 1; }       // workgroups per compute unit

template <int NS, int KH, bool DUAL, bool MASK>
__global__ __launch_bounds__(NS * 64, split_stream_held(NS, KH) * NS / 4) void gemm_split_stream_kernel(GemmArgs g, const uint16_t *Wt, uint32_t ku_total, uint32_t n_pad) {
    constexpr int CG = NS / KH, PLANE = 33, BUF = KH * 3 * 16 * PLANE * 16, CP = 36, NT = NS * 64;
    constexpr int RPP = NT / (16 * KH), NR = 32 / RPP;  // rows of A per pass, units of a thread in a tile
    constexpr int NP = 4 / KH;                          // a lane's 16-byte pieces of C in a tile
    __shared__ __attribute__((aligned(16))) char smem[split_stream_lds(NS, KH)];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = wave % CG, kh = wave / CG;           // the wave's columns and part of the reduction
    const int l32 = lane & 31, half = lane >> 5;
    const int n0 = static_cast<int>(blockIdx.y) * (CG * 32);
    float *slot0 = reinterpret_cast<float *>(smem + 2 * BUF) + cg * 32 * CP;
    float *bias = reinterpret_cast<float *>(smem + 2 * BUF + split_stream_slots(NS, KH) * 32 * CP * 4);
    const int64_t full = (g.M - 1) / 32;                // tiles before the one that holds the last row

    for (int c = tid; c < CG * 32; c += NT) bias[c] = (g.bias && n0 + c < g.N) ? g.bias[n0 + c] : 0.f;
    bf16x8 w[3][8];     // (a wave beyond the last column of the image holds its last columns: never stored)
    {
        const uint32_t col = n0 + cg * 32, n = col + 32 <= n_pad ? col : n_pad - 32;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const uint32_t u = 16 * kh + 2 * s;
                uint4 x = make_uint4(0u, 0u, 0u, 0u);
                if (u < ku_total)                       // (whole steps of 32 k: uniform)
                    x = *reinterpret_cast<const uint4 *>(Wt + ((static_cast<size_t>(p) * ku_total + u + half) * n_pad + n + l32) * 8);
                w[p][s] = __builtin_bit_cast(bf16x8, x);
            }
    }
    // the thread's unit of 8 k (rows r0, r0 + RPP ..): where it starts in tile 0, bytes from tile to tile, elements that exist
    const int v = tid % (16 * KH), r0 = tid / (16 * KH);
    const bool second = DUAL && 8 * v >= g.K1p;
    const int kk = second ? 8 * v - static_cast<int>(g.K1p) : 8 * v;
    const int64_t ld = second ? g.lda2 : g.lda;
    const int have = static_cast<int>(second ? g.K - g.K1p : DUAL ? g.K1 : g.K) - kk;
    const char *src = (second ? g.A2 : g.A) + (r0 * ld + (have > 0 ? kk : 0)) * 4;      // (units beyond the width read the first one and are cleared)
    const uint32_t tb = static_cast<uint32_t>(ld) * 128, at1 = have > 4 ? 16 : 0;
    const bool ragged = DUAL || g.K < 128 * KH;
    typedef float4 Rows[2 * NR];
    auto load = [&](int64_t t, Rows &r) __attribute__((always_inline)) {
        const char *p = src + static_cast<uint64_t>(static_cast<uint32_t>(t < full ? t : full - 1)) * tb;
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            r[2 * q] = *reinterpret_cast<const float4 *>(p + q * (tb / NR));
            r[2 * q + 1] = *reinterpret_cast<const float4 *>(p + (q * (tb / NR) + at1));
        }
    };
    auto load_last = [&](Rows &r) __attribute__((always_inline)) {            // the rows that exist, no further than their width
        const int rows = static_cast<int>(g.M - full * 32);
        const char *p = src + full * tb;
#pragma unroll
        for (int q = 0; q < NR; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int n = r0 + RPP * q < rows ? have - 4 * h : 0;
                r[2 * q + h] = load4<false>(p + q * (tb / NR), 4 * h, n < 4 ? n : 4, 1);
            }
    };
    auto clear = [&](Rows &r) __attribute__((always_inline)) {                // what lies beyond the width
        if (ragged)
#pragma unroll
            for (int q = 0; q < 2 * NR; ++q) {
                const int n = have - 4 * (q & 1);
                r[q] = make_float4(n > 0 ? r[q].x : 0.f, n > 1 ? r[q].y : 0.f, n > 2 ? r[q].z : 0.f, n > 3 ? r[q].w : 0.f);
            }
    };
    auto put = [&](Rows &r, char *As) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const float x[8] = {r[2 * q].x, r[2 * q].y, r[2 * q].z, r[2 * q].w, r[2 * q + 1].x, r[2 * q + 1].y, r[2 * q + 1].z, r[2 * q + 1].w};
            uint32_t u[4][3];
#pragma unroll
            for (int e = 0; e < 4; ++e) split3_pair(x[2 * e], x[2 * e + 1], u[e]);
#pragma unroll
            for (int p = 0; p < 3; ++p)
                *reinterpret_cast<uint4 *>(As + (((v / 16 * 3 + p) * 16 + v % 16) * PLANE + r0 + RPP * q) * 16) =
                    make_uint4(u[0][p], u[1][p], u[2][p], u[3][p]);
        }
    };
    // the lane's pieces of its wave's part of the result: columns col0 .. col0 + 3 of rows cr, cr + 8 ..
    const int cr = 16 * kh + lane / 8, c4 = 4 * (lane % 8), col0 = n0 + cg * 32 + c4;
    const uint32_t ldc4 = static_cast<uint32_t>(g.ldc) * 4, ldm4 = static_cast<uint32_t>(g.ldm) * 4;
    const bool whole = col0 + 4 <= g.N;
    const bool cut = g.N % 4 != 0;                      // a group of four columns ends inside the matrix (uniform)
    auto finish = [&](float x, float b) __attribute__((always_inline)) {
        x += b;
        return g.relu && !(x > 0.f) ? 0.f : x;
    };

    // rows: of the tile that exist; buf: the stage (and, for KH = 2, the slot) it uses; next: the rows that are cut meanwhile, into the
    // other stage, and then replaced by those of tile t_next, where there are more
    auto tile = [&](int64_t t, int rows, int buf, auto more, Rows &next, int64_t t_next) __attribute__((always_inline)) {
        const char *As = smem + buf * BUF + kh * 3 * 16 * PLANE * 16;
        float *slot = slot0 + (KH == 1 ? 0 : buf * CG * 32 * CP);
        float4 mk[NP];
        float rs[NP];
        if constexpr (MASK) {
            const char *mbase = g.mask + t * 32 * g.ldm * 4;
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int row = cr + 8 * p < rows ? cr + 8 * p : rows - 1;
                mk[p] = *reinterpret_cast<const float4 *>(mbase + (static_cast<uint32_t>(row) * ldm4 + (whole ? 4u * col0 : 0u)));
            }
        }
        if (g.rscale)
#pragma unroll
            for (int p = 0; p < NP; ++p) rs[p] = g.rscale[t * 32 + (cr + 8 * p < rows ? cr + 8 * p : rows - 1)];
        constexpr bool MORE = decltype(more)::value;
        if constexpr (MORE) clear(next);
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            bf16x8 x[3];
#pragma unroll
            for (int p = 0; p < 3; ++p)
                x[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(As + ((p * 16 + 2 * s + half) * PLANE + l32) * 16));
            // the six piece products, smallest first
#define CG_PIECES(PA_, PB_) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[PB_][s], x[PA_], acc, 0, 0, 0);
            CG_PIECES(2, 0) CG_PIECES(0, 2) CG_PIECES(1, 1) CG_PIECES(1, 0) CG_PIECES(0, 1) CG_PIECES(0, 0)
#undef CG_PIECES
        }
        if constexpr (MORE) put(next, smem + (buf ^ 1) * BUF);
        // the operands of one unit ahead of the matrix instructions, no more (the registers are the weights'); from the second unit on
        // the next rows are cut behind them, a few vector instructions each
        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s < 7) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (MORE && s > 0) __builtin_amdgcn_sched_group_barrier(0x002, NR == 1 ? 2 : 4, 0);
            }
            if (MORE && s > 0) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE) load(t_next, next);
        // registers 4 q ..: columns 8 q + 4 half .. of row l32.  KH = 2: first the rows that the other wave of these columns stores
        float4 *at = reinterpret_cast<float4 *>(&slot[l32 * CP + 4 * half]);
        if (KH == 1 || l32 / 16 != kh)
#pragma unroll
            for (int q = 0; q < 4; ++q) at[2 * q] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        if constexpr (KH == 2) {
            __syncthreads();
            if (l32 / 16 == kh)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 o = at[2 * q];
                    at[2 * q] = make_float4(acc[4 * q] + o.x, acc[4 * q + 1] + o.y, acc[4 * q + 2] + o.z, acc[4 * q + 3] + o.w);
                }
        }
        __builtin_amdgcn_wave_barrier();
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc(g.C + t * 32 * g.ldc * 4, 0, 0x7fffffff, 0x00027000);
        const float4 b4 = *reinterpret_cast<const float4 *>(&bias[cg * 32 + c4]);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            float4 x = *reinterpret_cast<const float4 *>(&slot[(cr + 8 * p) * CP + c4]);
            x = make_float4(finish(x.x, b4.x), finish(x.y, b4.y), finish(x.z, b4.z), finish(x.w, b4.w));
            if constexpr (MASK)
                x = make_float4(mk[p].x > 0.f ? x.x : 0.f, mk[p].y > 0.f ? x.y : 0.f, mk[p].z > 0.f ? x.z : 0.f, mk[p].w > 0.f ? x.w : 0.f);
            if (g.rscale) x = make_float4(x.x * rs[p], x.y * rs[p], x.z * rs[p], x.w * rs[p]);
            const uint32_t off = cr + 8 * p < rows && whole ? (cr + 8 * p) * ldc4 + 4u * col0 : 0xfffffff0u;
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rsrc, off, 0, 2);
        }
        if (cut) {
#pragma unroll 1
            for (int e = 0; e < 4 * NP; ++e) {
                const int row = cr + 8 * (e / 4), col = col0 + e % 4;
                const bool in = !whole && row < rows && col < g.N;
                float x = finish(slot[row * CP + c4 + e % 4], bias[cg * 32 + c4 + e % 4]);
                if constexpr (MASK) {
                    if (in && !(*reinterpret_cast<const float *>(g.mask + ((t * 32 + row) * g.ldm + col) * 4) > 0.f)) x = 0.f;
                }
                if (g.rscale && in) x *= g.rscale[t * 32 + row];
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), rsrc, in ? row * ldc4 + 4u * col : 0xfffffff0u, 0, 0);
            }
        }
        if constexpr (KH == 1) __syncthreads();
    };
    // as many dropped stores as the tiles before would have issued, so that the waits of the loop can allow for them
    auto dropped = [&](uint32_t at) __attribute__((always_inline)) {
        auto rsrc = __builtin_amdgcn_make_buffer_rsrc(g.C, 0, 0x7fffffff, 0x00027000);
#pragma unroll
        for (int p = 0; p < NP; ++p) __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, rsrc, at + 16 * p, 0, 2);
    };
    Rows ra, rb;
    const int64_t step = gridDim.x;
    int64_t t = blockIdx.x;
    if (t < full) {                                      // uniform over the workgroup
        load(t, ra);
        load(t + step, rb);
        dropped(0xffffff00u);
        clear(ra);
        put(ra, smem);
        load(t + 2 * step, ra);
        dropped(0xffffff40u);
        __syncthreads();
        for (; t + step < full; t += 2 * step) {         // (one way out: the waits are counted over every path)
            tile(t, 32, 0, std::true_type{}, rb, t + 3 * step);
            tile(t + step, 32, 1, std::true_type{}, ra, t + 4 * step);
        }
        if (t < full) {
            tile(t, 32, 0, std::false_type{}, ra, 0);
            t += step;
        }
        __syncthreads();                                 // stages and slots are free
    }
    if (t == full) {                                     // the tile with the last row (t went through every residue: one workgroup's)
        load_last(ra);
        put(ra, smem);
        __syncthreads();
        tile(t, static_cast<int>(g.M - full * 32), 0, std::false_type{}, ra, 0);
    }
}

// what the kernels for two products in one launch are told
struct SmallGemmArgs {
    GemmArgs g;                     // tile grid, sizes, epilogue; A2 / lda2 / K1 not used
    // second product of a sum C = A B + A2 B2 (dual), or second problem of the same shape C2 = A2 B2 (pair)
    const char *A2; int64_t lda2;
    const char *B2; int64_t ldb2;
    char *C2; int64_t ldc2;
    float *part2;
    const float *rscale2;
    int64_t K2;                     // of the dual form
    int64_t M2;                     // rows of the second problem
    int dual;
};

// The weight gradient X^T G in three pieces: both operands are stored across the reduction index (vertices), and nothing is staged.  A
// wave holds 128 x (TB * 32) results (TB = 4: all 256 accumulation registers) and loads both operands as the matrix instruction wants
// them: a lane eight vertices of one column, each load two rows of 32 columns.  It cuts the next operands between the matrix
// instructions, a pair of numbers behind every third of them, and asks for the numbers of the step after as soon as a pair is cut: no
// LDS, no barrier, one wave per SIMD with one step (16 KB) on its way.  The four waves of a workgroup take quarters of its vertices and add
// their results through LDS, in wave order, when a part ends: parts are as many as make the chains of fp32 additions no longer than one per
// split of the other kernels (choose_split), if longer than COLS_CHAIN (256 x 256 x 306000, error against fp64: one part 1.13e-6, two 8.2e-7,
// tiles staged through LDS 9.3e-7; a part more costs about 10 us there).
// Rows beyond the end of a wave's vertices are dropped by the buffer's bounds (zeros); columns beyond the operand's width only reach
// results that are not stored.  No alignment is asked for.  PMC at 256 x 256 x 306000: matrix cores busy 73 % of the time, at 1.76 GHz.
// us with the sum over parts, eight-wave tiles of 128 x 128 staged through LDS -> here: 256 x 256 x 306000 281 -> 217, 100 x 256 x
// 306000 188 -> 133, 602 x 256 x 180000 420 -> 298, 100 x 256 x 70001 53 -> 35, 602 x 200 x 30000 102 -> 60, 2000 x 1000 x 1000 135 -> 32.
constexpr int COLS_CHAIN = 512;
constexpr int COLS_PITCH = 72;      // floats per row of 64 results on their way through LDS (four rows further = other half of the banks)

template <int TB, bool SUMS>
__global__ __launch_bounds__(256, 1) void gemm_split_cols_kernel(SmallGemmArgs p2, int parts) {
    GemmArgs g = p2.g;
    if (blockIdx.y != 0) {                              // the second of a pair: another first operand, the same G
        g.A = p2.A2; g.lda = p2.lda2; g.C = p2.C2; g.ldc = p2.ldc2; g.part = p2.part2;
    }
    constexpr int TA = 4;
    __shared__ __attribute__((aligned(16))) float red[4][TA][32 * COLS_PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (g.S < NUM_XCD) {                                // too few splits for every L2 domain to have one: the tiles go to all of them
        const int tile = static_cast<int>(blockIdx.x) % (g.gx * g.gy);
        bz = static_cast<int>(blockIdx.x) / (g.gx * g.gy);
        bx = tile % g.gx;
        by = tile / g.gx;
    } else if (!tile_coords(g, &bx, &by, &bz)) {
        return;                                         // uniform over the workgroup
    }
    const int64_t m0 = static_cast<int64_t>(by) * (TA * 32), n0 = static_cast<int64_t>(bx) * (TB * 32);
    // the wave's vertices: `parts` stretches of g.k_chunk (a multiple of 32) one after the other
    const int64_t k_begin = (static_cast<int64_t>(bz) * 4 + wave) * parts * g.k_chunk;
    const int64_t k_have = g.K - k_begin < parts * g.k_chunk ? g.K - k_begin : parts * g.k_chunk;
    const int n_rows = k_have > 0 ? static_cast<int>(k_have) : 0;
    const int lda = static_cast<int>(g.lda) * 4, ldb = static_cast<int>(g.ldb) * 4;         // bytes
    const int width_a = static_cast<int>(g.M - m0 < TA * 32 ? g.M - m0 : TA * 32) * 4, width_b = static_cast<int>(g.N - n0 < TB * 32 ? g.N - n0 : TB * 32) * 4;
    const char *pa = g.A + (n_rows > 0 ? k_begin * lda + m0 * 4 : 0), *pb = g.B + (n_rows > 0 ? k_begin * ldb + n0 * 4 : 0);
    // the 16 rows from the wave's row `row` on, as many as there are
    auto rows16 = [&](const char *p, int ld, int row, int width) __attribute__((always_inline)) {
        const int n = n_rows - row < 16 ? n_rows - row : 16;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, n > 0 ? (n - 1) * ld + width : 0, 0x00027000);
    };
    uint32_t oa[8], ob[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        oa[j] = static_cast<uint32_t>(half * 8 + j) * lda + l32 * 4;
        ob[j] = static_cast<uint32_t>(half * 8 + j) * ldb + l32 * 4;
    }
    float ra[TA][8], rb[TB][8];                     // numbers of the step after next (ra[1 ..]: of the next)
    u32x4 ap[2][3], bp[2][TB][3];                   // pieces: of this tile of 32 rows and the next, of this step's columns and the next's
    floatx16 acc[TA][TB];
    double bsum[TB] = {};                           // SUMS: sums of the lane's columns of G
    float tsum = 0.f;
    auto load2 = [&](auto rsrc, const uint32_t (&o)[8], int tile, int e, float (&r)[8]) __attribute__((always_inline)) {
        r[2 * e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o[2 * e] + tile * 128, 0, 0));
        r[2 * e + 1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, o[2 * e + 1] + tile * 128, 0, 0));
    };
    auto cut2 = [&](const float (&r)[8], int e, u32x4 (&p)[3]) __attribute__((always_inline)) {
        uint32_t u[3];
        split3_pair(r[2 * e], r[2 * e + 1], u);
#pragma unroll
        for (int x = 0; x < 3; ++x) p[x][e] = u[x];
    };
    auto add_b = [&](int j, int e) __attribute__((always_inline)) {     // a step's eight numbers in fp32, the running sum a double
        if constexpr (SUMS) {
            const float t = rb[j][2 * e] + rb[j][2 * e + 1];
            tsum = e == 0 ? t : tsum + t;
            if (e == 3) bsum[j] += static_cast<double>(tsum);
        }
    };
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    clear();
    {
        auto sa = rows16(pa, lda, 0, width_a), sb = rows16(pb, ldb, 0, width_b);
        auto sa1 = rows16(pa + 16 * lda, lda, 16, width_a), sb1 = rows16(pb + 16 * ldb, ldb, 16, width_b);
#pragma unroll
        for (int e = 0; e < 4; ++e) load2(sa, oa, 0, e, ra[0]);
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) load2(sb, ob, j, e, rb[j]);
#pragma unroll
        for (int e = 0; e < 4; ++e) cut2(ra[0], e, ap[0]);
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                cut2(rb[j], e, bp[0][j]);
                add_b(j, e);
            }
        // in the order in which the loop asks for them: its waits are counted over both ways in
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                __builtin_amdgcn_sched_barrier(0);
                if (i + 1 < TA) load2(sa, oa, i + 1, e, ra[(i + 1) % TA]);
                else load2(sa1, oa, 0, e, ra[0]);
                if (i < TB) load2(sb1, ob, i, e, rb[i]);
            }
        __builtin_amdgcn_sched_barrier(0);
    }
    int row = 0;
    auto step = [&](auto parity) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value;
        pa += 16 * lda;
        pb += 16 * ldb;
        auto sa1 = rows16(pa, lda, row + 16, width_a), sa2 = rows16(pa + 16 * lda, lda, row + 32, width_a), sb2 = rows16(pb + 16 * ldb, ldb, row + 32, width_b);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < TA; ++i) {
            const int c = i & 1, ni = (i + 1) % TA, j2 = i % TB;
            const int groups = i < TB ? 8 : 4;          // pairs that are cut meanwhile: of the next 32 rows, and of 32 of the next step's columns
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (q >= groups) continue;
                const int e = groups == 8 ? q / 2 : q, first = 6 * TB * q / groups, last = 6 * TB * (q + 1) / groups;
#pragma unroll
                for (int m = 0; m < 6 * TB; ++m) {
                    if (m < first || m >= last) continue;
                    constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};       // the six piece products, smallest first
                    acc[i][m % TB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ap[c][PA[m / TB]]),
                                                                             __builtin_bit_cast(bf16x8, bp[P][m % TB][PB[m / TB]]), acc[i][m % TB], 0, 0, 0);
                }
                if (groups == 4 || q % 2 == 0) {
                    cut2(ra[ni], e, ap[c ^ 1]);
                    if (i + 1 < TA) load2(sa1, oa, ni, e, ra[ni]);
                    else load2(sa2, oa, ni, e, ra[ni]);
                } else {
                    cut2(rb[j2], e, bp[P ^ 1][j2]);
                    add_b(j2, e);
                    load2(sb2, ob, j2, e, rb[j2]);
                }
#pragma unroll
                for (int m = 0; m < 6 * TB; ++m) {
                    if (m < first || m >= last) continue;
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                // one matrix instruction
                    __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);                // vector instructions behind it
                    if (m > first) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0); // a load
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        row += 16;
    };
    static_assert(TA % 2 == 0 && TB <= TA, "a tile of columns is cut beside a tile of rows");
    for (int part = 0; part < parts; ++part) {
        const int end = static_cast<int>((part + 1) * g.k_chunk);
        while (row < end && row < n_rows) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
        const int z = bz * parts + part;
        int ln = lane;
        asm volatile("" : "+v"(ln));        // what follows from it is formed here: held through the loop it takes registers that are not there
        const int c32 = ln & 31, hf = ln >> 5;
        if constexpr (SUMS) {
            // (what the steps ahead have added belongs to the next part: the parts' sums are added up all the same)
            double (*bred)[TB * 32] = reinterpret_cast<double (*)[TB * 32]>(&red[0][0][0]);
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                bred[2 * wave + hf][j * 32 + c32] = bsum[j];
                bsum[j] = 0.0;
            }
            __syncthreads();
            const int col = 64 * wave + ln;
            if (by == 0 && blockIdx.y == 0 && col < TB * 32 && n0 + col < g.N) {
                double t = 0.0;
                for (int y = 0; y < 8; ++y) t += bred[y][col];
                g.colpart[z * g.N + n0 + col] = static_cast<float>(t);
            }
            __syncthreads();
        }
        // 64 columns at a time: the four waves' results side by side, then each wave adds up and stores 32 rows of them
#pragma unroll
        for (int h = 0; h < TB / 2; ++h) {
#pragma unroll
            for (int i = 0; i < TA; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) red[wave][i][(8 * (r >> 2) + 4 * hf + (r & 3)) * COLS_PITCH + j * 32 + c32] = acc[i][2 * h + j][r];
            __syncthreads();
            const int64_t col = n0 + h * 64 + 4 * (ln % 16);
            const bool vec = g.part ? g.N % 4 == 0 && reinterpret_cast<uintptr_t>(g.part) % 16 == 0
                                    : g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(g.C) % 16 == 0;
#pragma unroll 1
            for (int p = 0; p < 8; ++p) {
                const int lr = 4 * p + ln / 16;
                const int64_t at = m0 + wave * 32 + lr;
                float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float4 x = *reinterpret_cast<const float4 *>(&red[w][wave][lr * COLS_PITCH + 4 * (ln % 16)]);
                    v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
                }
                if (at >= g.M || col >= g.N) continue;
                float *dst = g.part ? g.part + (static_cast<int64_t>(z) * g.M + at) * g.N + col : reinterpret_cast<float *>(g.C) + at * g.ldc + col;
                if (!g.part)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < g.N) v[e] = epilogue_value(g, at, col + e, v[e]);
                if (vec && col + 4 <= g.N) {
                    *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < g.N) dst[e] = v[e];
                }
            }
            __syncthreads();
        }
        clear();
    }
}

// X^T G of bf16 operands in the same manner, bound by memory: a wave's 128 x (TB * 32) results, four (TB) columns of a vertex per lane and
// load, so tile i of 32 rows holds the columns 4 r + i of X; eight vertices of a column come together by byte permutes.  Three steps of 16
// vertices (8 KB each) are on their way while one is multiplied.  The waves of all splits take steps in turn, so that what is read at any
// time is one stretch of the operands (a stretch per wave: 256 x 256 x 980000 241 us instead of 228, 128 x 256 167 instead of 152).  Rows start on
// 16 bytes; a last row that ends inside a group of four columns is read apart, column by column.
// us with the sum over parts, tiles staged through LDS or gemm_small_kernel -> here: 256 x 256 x 980000 320 -> 228 (4.6 TB/s), 128 x 256 x 980000 191 -> 152, 256 x 47 x
// 980000 146 -> 112, 389 x 200 x 98712 84 -> 61, 602 x 256 x 30000 47 -> 32, 200 x 2 x 98712 29 -> 19, 100 x 16 x 250000 41 -> 21.
template <int TB, bool SUMS>
__global__ __launch_bounds__(256, 1) void gemm_bf16_cols_kernel(SmallGemmArgs p2, int parts) {
    GemmArgs g = p2.g;
    if (blockIdx.y != 0) {                              // the second of a pair: another first operand, the same G
        g.A = p2.A2; g.lda = p2.lda2; g.C = p2.C2; g.ldc = p2.ldc2; g.part = p2.part2;
    }
    constexpr int TA = 4, AHEAD = 4, CP = TB * 32 + 4;         // steps held, floats per row of the wave's results on their way through LDS
    constexpr int WB = TB / 2;                                 // dwords of a lane's columns of G
    __shared__ __attribute__((aligned(16))) float red[4][64 * CP];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (g.S < NUM_XCD) {                                // too few splits for every L2 domain to have one: the tiles go to all of them
        const int tile = static_cast<int>(blockIdx.x) % (g.gx * g.gy);
        bz = static_cast<int>(blockIdx.x) / (g.gx * g.gy);
        bx = tile % g.gx;
        by = tile / g.gx;
    } else if (!tile_coords(g, &bx, &by, &bz)) {
        return;                                         // uniform over the workgroup
    }
    const int64_t m0 = static_cast<int64_t>(by) * (TA * 32), n0 = static_cast<int64_t>(bx) * (TB * 32);
    const bool ragged = (g.M | g.N) % 4 != 0;           // the matrices' last row (there is one: g.K > 0) is read apart
    const int64_t k_all = ragged ? g.K - 1 : g.K;
    const int k_first = (bz * 4 + wave) * 16, k_step = 64 * g.S, n_all = static_cast<int>(k_all);
    const int lda = static_cast<int>(g.lda) * 2, ldb = static_cast<int>(g.ldb) * 2;         // bytes
    const int left_a = static_cast<int>(g.M - m0 < TA * 32 ? g.M - m0 : TA * 32), left_b = static_cast<int>(g.N - n0 < TB * 32 ? g.N - n0 : TB * 32);
    const int width_a = (left_a + 3) / 4 * 8, width_b = (left_b + 3) / 4 * 8;
    const char *pa = g.A + (static_cast<int64_t>(k_first) * lda + m0 * 2), *pb = g.B + (static_cast<int64_t>(k_first) * ldb + n0 * 2);
    auto rows16 = [&](const char *p, int ld, int row, int width) __attribute__((always_inline)) {
        const int n = n_all - row < 16 ? n_all - row : 16;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), 0, n > 0 ? (n - 1) * ld + width : 0, 0x00027000);
    };
    uint32_t oa[8], ob[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        oa[j] = static_cast<uint32_t>(half * 8 + j) * lda + l32 * 8;
        ob[j] = static_cast<uint32_t>(half * 8 + j) * ldb + l32 * (2 * TB);
    }
    struct Raw { uint32_t a[8][2], b[8][WB]; };
    Raw raw[AHEAD];
    u32x4 oa4[2][TA], ob4[2][TB];                       // operands of this step and the next
    floatx16 acc[TA][TB];
    double bsum[TB] = {};
    int row = k_first;                                        // of the step that is asked for next
    auto ask = [&](Raw &r) __attribute__((always_inline)) {
        auto sa = rows16(pa, lda, row, width_a), sb = rows16(pb, ldb, row, width_b);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(sa, oa[j], 0, 0));
            r.a[j][0] = v.x; r.a[j][1] = v.y;
            if constexpr (WB == 2) {
                const u32x2 w = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(sb, ob[j], 0, 0));
                r.b[j][0] = w.x; r.b[j][WB - 1] = w.y;
            } else {
                r.b[j][0] = __builtin_amdgcn_raw_buffer_load_b32(sb, ob[j], 0, 0);
            }
        }
        pa += static_cast<int64_t>(k_step) * lda;
        pb += static_cast<int64_t>(k_step) * ldb;
        row += k_step;
    };
    // eight vertices of each of the lane's columns
    auto turn = [&](const Raw &r, u32x4 (&a)[TA], u32x4 (&b)[TB]) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int i = 0; i < TA; ++i)
                a[i][e] = __builtin_amdgcn_perm(r.a[2 * e + 1][i / 2], r.a[2 * e][i / 2], i & 1 ? 0x07060302u : 0x05040100u);
#pragma unroll
            for (int j = 0; j < TB; ++j)
                b[j][e] = __builtin_amdgcn_perm(r.b[2 * e + 1][j / 2], r.b[2 * e][j / 2], j & 1 ? 0x07060302u : 0x05040100u);
        }
        if constexpr (SUMS) {                           // a step's eight numbers in fp32, the running sum a double
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                float t = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) t += __uint_as_float(b[j][e] << 16) + __uint_as_float(b[j][e] & 0xffff0000u);
                bsum[j] += static_cast<double>(t);
            }
        }
    };
    auto multiply = [&](const u32x4 (&a)[TA], const u32x4 (&b)[TB]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
    };
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    };
    clear();
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
        ask(raw[p]);
        __builtin_amdgcn_sched_barrier(0);
    }
    turn(raw[0], oa4[0], ob4[0]);
    ask(raw[0]);
    int at = 0;                                         // rows multiplied
    for (int part = 0; part < parts; ++part) {
        const int end = static_cast<int>((part + 1) * g.k_chunk);
        while (at < end) {               // (g.k_chunk: a multiple of AHEAD steps)
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) {
                multiply(oa4[p & 1], ob4[p & 1]);
                turn(raw[(p + 1) % AHEAD], oa4[(p & 1) ^ 1], ob4[(p & 1) ^ 1]);
                ask(raw[(p + 1) % AHEAD]);
                __builtin_amdgcn_sched_barrier(0);
            }
            at += 16 * AHEAD;
        }
        if (ragged && bz == 0 && wave == 0 && part == 0) {
            Raw r{};
            const uint16_t *xa = reinterpret_cast<const uint16_t *>(g.A) + (g.K - 1) * g.lda + m0 + 4 * l32;
            const uint16_t *xb = reinterpret_cast<const uint16_t *>(g.B) + (g.K - 1) * g.ldb + n0 + TB * l32;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (half == 0 && 4 * l32 + e < left_a) r.a[0][e / 2] |= static_cast<uint32_t>(xa[e]) << (16 * (e & 1));
#pragma unroll
            for (int e = 0; e < TB; ++e)
                if (half == 0 && TB * l32 + e < left_b) r.b[0][e / 2] |= static_cast<uint32_t>(xb[e]) << (16 * (e & 1));
            u32x4 ta[TA], tb[TB];
            turn(r, ta, tb);
            multiply(ta, tb);
        }
        const int z = bz * parts + part;
        int ln = lane;
        asm volatile("" : "+v"(ln));        // what follows from it is formed here: held through the loop it takes registers
        const int c32 = ln & 31, hf = ln >> 5;
        if constexpr (SUMS) {
            // (what the step ahead has added belongs to the next part: the parts' sums are added up all the same)
            double (*bred)[TB * 32] = reinterpret_cast<double (*)[TB * 32]>(&red[0][0]);
#pragma unroll
            for (int j = 0; j < TB; ++j) {
                bred[2 * wave + hf][TB * c32 + j] = bsum[j];
                bsum[j] = 0.0;
            }
            __syncthreads();
            const int col = 64 * wave + ln;
            if (by == 0 && blockIdx.y == 0 && col < TB * 32 && n0 + col < g.N) {
                double t = 0.0;
                for (int y = 0; y < 8; ++y) t += bred[y][col];
                g.colpart[z * g.N + n0 + col] = static_cast<float>(t);
            }
            __syncthreads();
        }
        // two tiles of 32 rows at a time: the four waves' results side by side, then each wave adds up and stores 16 rows of them
#pragma unroll
        for (int h = 0; h < TA / 2; ++h) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float *to = &red[wave][(2 * (8 * (r >> 2) + 4 * hf + (r & 3)) + i) * CP + TB * c32];
#pragma unroll
                    for (int j = 0; j < TB; ++j) to[j] = acc[2 * h + i][j][r];
                }
            __syncthreads();
            constexpr int CGS = TB * 8, RPP = 64 / CGS;          // groups of four columns in a row, rows per pass
            const int64_t col = n0 + 4 * (ln % CGS);
            const bool vec = g.part ? g.N % 4 == 0 && reinterpret_cast<uintptr_t>(g.part) % 16 == 0
                                    : g.ldc % 4 == 0 && reinterpret_cast<uintptr_t>(g.C) % 16 == 0;
#pragma unroll 1
            for (int p = 0; p < 16 / RPP; ++p) {
                const int lr = 16 * wave + RPP * p + ln / CGS;           // row 2 r + i: column 4 r + 2 h + i of X
                const int64_t to = m0 + 4 * (lr / 2) + 2 * h + lr % 2;
                float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float4 x = *reinterpret_cast<const float4 *>(&red[w][lr * CP + 4 * (ln % CGS)]);
                    v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
                }
                if (to >= g.M || col >= g.N) continue;
                if (!g.part) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < g.N) v[e] = epilogue_value(g, to, col + e, v[e]);
                    if (g.out_bf16) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (col + e < g.N) reinterpret_cast<uint16_t *>(g.C)[to * g.ldc + col + e] = static_cast<uint16_t>(f32_to_bf16_rne(v[e]));
                        continue;
                    }
                }
                float *dst = g.part ? g.part + (static_cast<int64_t>(z) * g.M + to) * g.N + col : reinterpret_cast<float *>(g.C) + to * g.ldc + col;
                if (vec && col + 4 <= g.N) {
                    *reinterpret_cast<float4 *>(dst) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < g.N) dst[e] = v[e];
                }
            }
            __syncthreads();
        }
        clear();
    }
}

// ---------------------------------------------------------------------------------------------------
// Small products, whose tiles of 128 rows would leave most of the chip idle and pay a round trip to memory per 16 or 32 k:
// here a workgroup owns 32 x (TN * 32) outputs, its four waves take quarters of the reduction (or, of a sum of two
// products, two waves each), and every wave loads its operands straight into the registers the matrix instruction reads
// them from, four units (fp32: 32 k, bf16: 64 k) at a time and one batch ahead: one or two round trips in all.  The four
// partial tiles are added through LDS in wave order.  No alignment is needed; k may be assigned to the instruction's k slots
// in any order as long as both operands agree, so a lane takes four (eight) consecutive k of its row.

// One unit of an operand: 4 fp32 k (of a half wave's 8) or 8 bf16 k (of 16), of one row / column of the result.
template <bool BF16> struct SmallUnit { float v[4]; };
template <> struct SmallUnit<true> { uint32_t v[4]; };

// ALONG: the operand is stored along the reduction index.  p: address of its first element at k = 0; step: bytes from one k
// to the next when not ALONG; the unit starts at k; elements from k_end on are zero (FULL: there are none).
template <bool BF16, bool ALONG, bool FULL>
__device__ __forceinline__ void small_load(const char *p, int64_t step, int64_t k, int64_t k_end, bool vec, SmallUnit<BF16> &r) {
    constexpr int ES = BF16 ? 2 : 4, NE = BF16 ? 8 : 4;
    if constexpr (ALONG) {
        if (FULL && vec) {
            const uint4 q = *reinterpret_cast<const uint4 *>(p + k * ES);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (BF16) r.v[e] = w[e];
                else r.v[e] = __uint_as_float(w[e]);
            }
            return;
        }
    }
    const int64_t d = ALONG ? ES : step;
    const char *q = p + k * d;
#pragma unroll
    for (int e = 0; e < NE; e += BF16 ? 2 : 1) {
        if constexpr (BF16) {
            const uint32_t lo = FULL || k + e < k_end ? *reinterpret_cast<const uint16_t *>(q + e * d) : 0u;
            const uint32_t hi = FULL || k + e + 1 < k_end ? *reinterpret_cast<const uint16_t *>(q + (e + 1) * d) : 0u;
            r.v[e / 2] = lo | (hi << 16);
        } else {
            r.v[e] = FULL || k + e < k_end ? *reinterpret_cast<const float *>(q + e * d) : 0.f;
        }
    }
}

constexpr int SMALL_UNITS = 4;      // units per batch
template <bool BF16> constexpr int SMALL_UNIT_K = BF16 ? 16 : 8;

// HOLD: epilogue operands held through the loop; in reductions over vertices, which hold none, registers for two waves per SIMD
// (see launch_small)
// (LDS of a workgroup: the four partial tiles, and the partial column sums)
template <int TN> struct SmallShared {
    static constexpr int PITCH = TN * 32 + 4;
    float red[4][32][PITCH];
    double bred[4][TN * 32];
};

template <bool BF16, bool A_KC, bool B_KC, int TN, bool HOLD>
__device__ __forceinline__ void small_tile(const SmallGemmArgs &s, SmallShared<TN> &lds, int64_t block, bool second) {
    constexpr int ES = BF16 ? 2 : 4, UK = SMALL_UNIT_K<BF16>, HK = UK / 2, UB = SMALL_UNITS;
    auto &red = lds.red;
    auto &bred = lds.bred;
    const GemmArgs &g = s.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (!tile_coords(g, block, &bx, &by, &bz)) return;      // uniform over the workgroup; second: the other problem of a pair
    const int64_t M = second ? s.M2 : g.M;
    const int64_t m0 = static_cast<int64_t>(by) * 32, n0 = static_cast<int64_t>(bx) * (TN * 32);
    // the wave's operands and its range of the reduction
    const bool alt = second || (s.dual && wave >= 2);
    const char *A = alt ? s.A2 : g.A, *B = alt ? s.B2 : g.B;
    const int64_t lda = alt ? s.lda2 : g.lda, ldb = alt ? s.ldb2 : g.ldb;
    int64_t k_end, k;
    if (s.dual) {
        const int64_t K = wave >= 2 ? s.K2 : g.K, per = (K + 2 * UK - 1) / (2 * UK) * UK;
        k = (wave & 1) * per;
        k_end = k + per < K ? k + per : K;
    } else {
        const int64_t per = g.k_chunk / 4;           // whole units
        k = bz * g.k_chunk + wave * per;
        k_end = k + per < g.K ? k + per : g.K;
    }
    // rows and columns beyond the matrices repeat the last one: what they give is never stored
    if (m0 >= M) return;                             // uniform over the workgroup
    const int64_t row = m0 + l32 < M ? m0 + l32 : M - 1;
    const char *pa = A + (A_KC ? row * lda : row) * ES;
    const char *pb[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int64_t c = n0 + j * 32 + l32, col = c < g.N ? c : g.N - 1;
        pb[j] = B + (B_KC ? col * ldb : col) * ES;
    }
    const int64_t sa = lda * ES, sb = ldb * ES;
    const bool va = (reinterpret_cast<uintptr_t>(A) | static_cast<uintptr_t>(sa)) % 16 == 0;
    const bool vb = (reinterpret_cast<uintptr_t>(B) | static_cast<uintptr_t>(sb)) % 16 == 0;

    SmallUnit<BF16> a[UB], b[UB][TN];
    auto fetch = [&](int64_t kb) __attribute__((always_inline)) {
        if (kb + UB * UK <= k_end) {
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int64_t ku = kb + u * UK + half * HK;
                small_load<BF16, A_KC, true>(pa, sa, ku, k_end, va, a[u]);
#pragma unroll
                for (int j = 0; j < TN; ++j) small_load<BF16, B_KC, true>(pb[j], sb, ku, k_end, vb, b[u][j]);
            }
        } else {
            // (a plain product's wave has a batch or little more: its whole units take the whole loads; element by element 10000 x 64 x 64
            // fp32 by W^T 13.1 us, so 10.3; 6000 x 128 x 128 bf16 9.3, so 6.7)
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const int64_t ku = kb + u * UK + half * HK;
                if (A_KC && kb + (u + 1) * UK <= k_end) {
                    small_load<BF16, A_KC, true>(pa, sa, ku, k_end, va, a[u]);
#pragma unroll
                    for (int j = 0; j < TN; ++j) small_load<BF16, B_KC, true>(pb[j], sb, ku, k_end, vb, b[u][j]);
                } else if (A_KC && kb + u * UK >= k_end) {
                    a[u] = SmallUnit<BF16>{};
#pragma unroll
                    for (int j = 0; j < TN; ++j) b[u][j] = SmallUnit<BF16>{};
                } else {
                    small_load<BF16, A_KC, false>(pa, sa, ku, k_end, va, a[u]);
#pragma unroll
                    for (int j = 0; j < TN; ++j) small_load<BF16, B_KC, false>(pb[j], sb, ku, k_end, vb, b[u][j]);
                }
            }
        }
    };
    floatx16 acc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
    // what the epilogue reads (clamped places): four columns per thread and pass, asked for ahead of the operands (HOLD), else ahead of
    // the exchange through LDS; reductions over vertices, which mostly write parts, ask for it element by element (see below)
    constexpr int PASSES = TN;                       // of 256 threads x 4 columns over 32 rows
    constexpr int ER = 256 / (TN * 8);
    int er = threadIdx.x / (TN * 8), ec = 4 * (threadIdx.x % (TN * 8));
    if constexpr (A_KC && !HOLD) {                   // (not worth registers in the loop)
        int tid = threadIdx.x;
        asm("" : "+v"(tid));
        er = tid / (TN * 8);
        ec = 4 * (tid % (TN * 8));
    }
    float *part = second ? s.part2 : g.part;
    char *C = second ? s.C2 : g.C;
    const int64_t ldc = second ? s.ldc2 : g.ldc;
    const float *rscale = second ? s.rscale2 : g.rscale;
    float e_c[PASSES][4], e_b[4], e_m[PASSES][4], e_s[PASSES];
    auto fetch_epilogue = [&]() __attribute__((always_inline)) {
        if (part) return;                            // uniform over the grid, as are the conditions below
        auto ccol = [&](int e) { return n0 + ec + e < g.N ? n0 + ec + e : g.N - 1; };
        auto crow = [&](int p) { return m0 + er + p * ER < M ? m0 + er + p * ER : M - 1; };
        if (g.bias)
#pragma unroll
            for (int e = 0; e < 4; ++e) e_b[e] = g.bias[ccol(e)];
        if (g.accumulate)
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) e_c[p][e] = epilogue_load(C, crow(p) * ldc + ccol(e), g.out_bf16);
        if (g.mask)
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
#pragma unroll
                for (int e = 0; e < 4; ++e) e_m[p][e] = epilogue_load(g.mask, crow(p) * g.ldm + ccol(e), g.mask_bf16);
        if (rscale)
#pragma unroll
            for (int p = 0; p < PASSES; ++p) e_s[p] = rscale[crow(p)];
    };
    if constexpr (A_KC && HOLD) fetch_epilogue();
    // column sums of B: the bias gradient rides on the weight gradient that reads dZ anyway.  However long a split is, a thread
    // adds no more than the 16 .. 32 terms of a step in fp32; its running sum and those of the workgroup are doubles.
    const bool sums = !A_KC && !B_KC && g.colpart && by == 0 && !second;      // uniform over the workgroup
    double bsum[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bsum[j] = 0.0;
    if (k < k_end) fetch(k);
    for (; k < k_end; k += UB * UK) {
        SmallUnit<BF16> ca[UB], cb[UB][TN];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
            ca[u] = a[u];
#pragma unroll
            for (int j = 0; j < TN; ++j) cb[u][j] = b[u][j];
        }
        if (k + UB * UK < k_end) fetch(k + UB * UK);
        if (sums) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                float t = 0.f;
#pragma unroll
                for (int u = 0; u < UB; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (BF16) t += __uint_as_float(cb[u][j].v[e] << 16) + __uint_as_float(cb[u][j].v[e] & 0xffff0000u);
                        else t += cb[u][j].v[e];
                    }
                bsum[j] += static_cast<double>(t);
            }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (BF16) {
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ca[u]), __builtin_bit_cast(bf16x8, cb[u][j]),
                                                                     acc[j], 0, 0, 0);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ca[u].v[e], cb[u][j].v[e], acc[j], 0, 0, 0);
                }
            }
    }
    if constexpr (A_KC && !HOLD) fetch_epilogue();
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[wave][8 * (r >> 2) + 4 * half + (r & 3)][j * 32 + l32] = acc[j][r];
    if (sums) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const double t = bsum[j] + __shfl_xor(bsum[j], 32);
            if (half == 0) bred[wave][j * 32 + l32] = t;
        }
    }
    __syncthreads();
    if (sums)
        for (int c = threadIdx.x; c < TN * 32; c += 256)
            if (n0 + c < g.N) g.colpart[bz * g.N + n0 + c] = static_cast<float>((bred[0][c] + bred[1][c]) + (bred[2][c] + bred[3][c]));
    if constexpr (!A_KC) {
        // four columns per thread, in an epilogue of its own: the pass below changes how the compiler orders the loads and waits of these
        // kernels' loops (bf16 weight gradients: 602 x 32 x 30000 45.9 us by it, 24.8 so; pairs of 100 x 200 x 66498 62, 50)
        for (int i = threadIdx.x; i < 32 * TN * 8; i += 256) {
            const int r = i / (TN * 8), c4 = i % (TN * 8);
            const int64_t orow = m0 + r, ocol = n0 + 4 * c4;
            if (orow >= M || ocol >= g.N) continue;
            float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float4 q = *reinterpret_cast<const float4 *>(&red[w][r][4 * c4]);
                v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
            }
            const int nv = g.N - ocol < 4 ? static_cast<int>(g.N - ocol) : 4;
            if (part) {
                float *o = part + (bz * M + orow) * g.N + ocol;
                for (int e = 0; e < nv; ++e) o[e] = v[e];
                continue;
            }
            for (int e = 0; e < nv; ++e) {
                const int64_t at = orow * ldc + ocol + e;
                float x = v[e];
                if (g.accumulate) x += epilogue_load(C, at, g.out_bf16);
                if (g.bias) x += g.bias[ocol + e];
                if (g.relu) x = x > 0.f ? x : 0.f;
                if (g.mask && !(epilogue_load(g.mask, orow * g.ldm + ocol + e, g.mask_bf16) > 0.f)) x = 0.f;
                if (rscale) x *= rscale[orow];
                if (g.out_bf16) reinterpret_cast<uint16_t *>(C)[at] = static_cast<uint16_t>(f32_to_bf16_rne(x));
                else reinterpret_cast<float *>(C)[at] = x;
            }
        }
        return;
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int r = er + p * ER;
        const int64_t orow = m0 + r, ocol = n0 + ec;
        if (orow >= M || ocol >= g.N) continue;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 q = *reinterpret_cast<const float4 *>(&red[w][r][ec]);
            v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
        }
        if (!part) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (g.accumulate) v[e] += e_c[p][e];
                if (g.bias) v[e] += e_b[e];
                if (g.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
                if (g.mask) v[e] = e_m[p][e] > 0.f ? v[e] : 0.f;
                if (rscale) v[e] *= e_s[p];
            }
        }
        float *o = part ? part + (bz * M + orow) * g.N + ocol : reinterpret_cast<float *>(C) + orow * ldc + ocol;
        uint16_t *ob = reinterpret_cast<uint16_t *>(C) + orow * ldc + ocol;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (ocol + e < g.N) {
                if (!part && g.out_bf16) ob[e] = static_cast<uint16_t>(f32_to_bf16_rne(v[e]));
                else o[e] = v[e];
            }
    }
}

template <bool BF16, bool A_KC, bool B_KC, int TN, bool HOLD>
__global__ __launch_bounds__(256, !A_KC && HOLD ? 2 : 1) void gemm_small_kernel(SmallGemmArgs s) {
    __shared__ __attribute__((aligned(16))) SmallShared<TN> lds;
    small_tile<BF16, A_KC, B_KC, TN, HOLD>(s, lds, blockIdx.x, blockIdx.y != 0);
}

// The products of a layer's backward pass that do not wait for one another, the weight gradients X^T G (column tiles of TW) and the input gradient
// G W^T (TX), in one launch: each alone leaves most of the chip idle and costs a launch.  Task i has the workgroups [first[i], first[i + 1]), the
// two problems of a pair one after the other.
struct SmallBatchArgs {
    SmallGemmArgs task[3];
    int first[4], nx[3], plain[3];
};
template <bool BF16, int TW, int TX>
__global__ __launch_bounds__(256, 2) void gemm_small_batch_kernel(SmallBatchArgs b) {
    __shared__ __attribute__((aligned(16))) union { SmallShared<TW> w; SmallShared<TX> x; } lds;
    const int wg = blockIdx.x, i = wg < b.first[1] ? 0 : wg < b.first[2] ? 1 : 2;
    const int at = wg - b.first[i], second = at >= b.nx[i];
    if (b.plain[i]) small_tile<BF16, true, true, TX, true>(b.task[i], lds.x, at - second * b.nx[i], second != 0);
    else small_tile<BF16, false, false, TW, BF16 && TW == 1>(b.task[i], lds.w, at - second * b.nx[i], second != 0);
}

// Reductions over vertices with a narrow second operand, C = A^T B, A [K x M] and B [K x N <= 64] in float, on the fp32 instruction
// (v_mfma_f32_16x16x4_f32): many more bytes than products, so memory bounds it.  An operand stored across the reduction index already
// lies as the instruction wants it when rows of the result are dealt to tiles in steps of four: a lane's 16-byte load of A, four
// neighbouring columns of row k, is its operand of four tiles.  So nothing is staged: a wave owns 128 x 16 NT results, loads four k
// at a time, NARROW_AHEAD batches ahead, and multiplies; the four waves of a workgroup take turns at the k of its split and are summed
// through LDS in wave order, splits by gemm_reduce_kernel.  Rows need no alignment.
constexpr int NARROW_AHEAD = 4;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_dword __attribute__((ext_vector_type(4), aligned(4)));

// A pair of problems of one shape (A2, B2, part2) runs as the second row of the grid.
template <int NT>
__global__ __launch_bounds__(256, NT <= 2 ? 3 : 2) void gemm_narrow_kernel(SmallGemmArgs p2) {
    GemmArgs &g = p2.g;
    const bool second = blockIdx.y != 0;
    if (second) { g.A = p2.A2; g.lda = p2.lda2; g.B = p2.B2; g.ldb = p2.ldb2; g.part = p2.part2; }
    constexpr int AHEAD = NARROW_AHEAD;
    __shared__ __attribute__((aligned(16))) f32x4 red[4][4 * NT][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quarter = lane >> 4;      // the lane's row / column of a tile, its k of a batch
    int bx, by, bz;
    if (!tile_coords(g, &bx, &by, &bz)) return;          // uniform over the workgroup
    const int64_t m0 = static_cast<int64_t>(by) * 128;
    const int64_t k_begin = static_cast<int64_t>(bz) * g.k_chunk;
    const int64_t k_end = k_begin + g.k_chunk < g.K ? k_begin + g.k_chunk : g.K;
    const float *A = reinterpret_cast<const float *>(g.A), *B = reinterpret_cast<const float *>(g.B);
    // columns beyond the matrices read others: what they give is never stored
    int64_t am[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int64_t m = m0 + 64 * u + 4 * l16;
        am[u] = m < g.M ? m : g.M - 1;
    }
    int bn[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) bn[j] = 16 * j + l16 < g.N ? 16 * j + l16 : static_cast<int>(g.N) - 1;

    f32x4 acc[2][4][NT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[u][c][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // column sums of B (see gemm_small_kernel): a lane adds AHEAD terms in fp32
    const bool sums = g.colpart && by == 0 && !second;
    double bsum[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) bsum[j] = 0.0;
    auto multiply = [&](const f32x4 (&a)[2], const float (&b)[NT]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[u][c][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][c], b[j], acc[u][c][j], 0, 0, 0);
    };
    // batches whose loads may run past the width of a row: 16 bytes of a row before the last three stay inside the matrix
    const int64_t first = k_begin + 4 * wave, limit = k_end < g.K - 3 ? k_end : g.K - 3;
    const int n = limit >= first + 4 ? static_cast<int>((limit - 4 - first) / 16 + 1) : 0;
    if (n > 0) {
        f32x4 a[AHEAD][2];
        float b[AHEAD][NT];
        const float *pa = A + (first + quarter) * g.lda, *pb = B + (first + quarter) * g.ldb;
        auto fetch = [&](int s, int p) __attribute__((always_inline)) {      // (after the last batch: that one again)
            const int64_t t = 16 * static_cast<int64_t>(s < n ? s : n - 1);
#pragma unroll
            for (int u = 0; u < 2; ++u) a[p][u] = *reinterpret_cast<const f32x4_dword *>(pa + t * g.lda + am[u]);
#pragma unroll
            for (int j = 0; j < NT; ++j) b[p][j] = pb[t * g.ldb + bn[j]];
        };
#pragma unroll
        for (int p = 0; p < AHEAD; ++p) fetch(p, p);
        int s = 0;
        for (; s + AHEAD <= n; s += AHEAD) {
            float t[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) t[j] = 0.f;
#pragma unroll
            for (int p = 0; p < AHEAD; ++p) {
                multiply(a[p], b[p]);
#pragma unroll
                for (int j = 0; j < NT; ++j) t[j] += b[p][j];
                fetch(s + p + AHEAD, p);
            }
            if (sums)
#pragma unroll
                for (int j = 0; j < NT; ++j) bsum[j] += static_cast<double>(t[j]);
        }
#pragma unroll
        for (int p = 0; p < AHEAD; ++p)
            if (s + p < n) {
                multiply(a[p], b[p]);
                if (sums)
#pragma unroll
                    for (int j = 0; j < NT; ++j) bsum[j] += static_cast<double>(b[p][j]);
            }
    }
    for (int64_t k = first + 16 * static_cast<int64_t>(n); k < k_end; k += 16) {      // what is left, element by element
        const int64_t row = k + quarter;
        f32x4 a[2];
        float b[NT];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int64_t m = m0 + 64 * u + 4 * l16 + c;
                a[u][c] = row < k_end && m < g.M ? A[row * g.lda + m] : 0.f;
            }
#pragma unroll
        for (int j = 0; j < NT; ++j) b[j] = row < k_end && 16 * j + l16 < g.N ? B[row * g.ldb + 16 * j + l16] : 0.f;
        multiply(a, b);
        if (sums)
#pragma unroll
            for (int j = 0; j < NT; ++j) bsum[j] += static_cast<double>(b[j]);
    }
    if (sums) {
        double (*bred)[NT * 16] = reinterpret_cast<double (*)[NT * 16]>(red);        // [16 groups of lanes][columns]
#pragma unroll
        for (int j = 0; j < NT; ++j) bred[4 * wave + quarter][16 * j + l16] = bsum[j];
        __syncthreads();
        const int c = threadIdx.x;
        if (c < NT * 16 && c < g.N) {
            double t = 0.0;
            for (int y = 0; y < 16; ++y) t += bred[y][c];
            g.colpart[bz * g.N + c] = static_cast<float>(t);
        }
    }
    // every wave adds up the tiles (u, wave, j) of all four, in wave order.  Register r of tile (u, c, j): row 64 u + 16 quarter +
    // 4 r + c, column 16 j + l16
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int j = 0; j < NT; ++j) red[wave][c * NT + j][lane] = acc[u][c][j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            f32x4 t = red[0][wave * NT + j][lane];
#pragma unroll
            for (int w = 1; w < 4; ++w) t += red[w][wave * NT + j][lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t m = m0 + 64 * u + 16 * quarter + 4 * r + wave;
                if (m < g.M && 16 * j + l16 < g.N) g.part[(static_cast<int64_t>(bz) * g.M + m) * g.N + 16 * j + l16] = t[r];
            }
        }
    }
}

// Plain fp32 products in three pieces whose 64 x 64 tiles are few for the chip or whose reduction is long for its tiles: a workgroup owns one tile and its
// four waves take quarters of the reduction, each for itself: operands go from memory straight into the registers of the matrix instruction,
// two steps of 16 k ahead, and are cut there; no barrier until the four partial tiles are added through LDS, in wave order.  Of 32 k a
// lane takes 16 neighbouring ones of its row, so that the loads that share a line of A follow one another.  Also the sum of two products (DUAL: the
// steps of the second follow those of the first) and two products of one shape (blockIdx.y, see SmallGemmArgs).  Rows need no alignment.
template <bool B_KC, bool DUAL>
__global__ __launch_bounds__(256, 2) void gemm_split_quarters_kernel(SmallGemmArgs p2) {
    constexpr int TM = 2, TN = 2, PITCH = 68;
    __shared__ __attribute__((aligned(16))) float red[4][64][PITCH];
    const GemmArgs &g = p2.g;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (!tile_coords(g, &bx, &by, &bz)) return;      // uniform over the workgroup
    const bool other = !DUAL && blockIdx.y != 0;     // the second of a pair
    const int64_t M = other ? p2.M2 : g.M;
    const int64_t m0 = static_cast<int64_t>(by) * 64, n0 = static_cast<int64_t>(bx) * 64;
    if (m0 >= M) return;
    struct Side { const char *a, *b; int64_t lda, ldb; bool va, vb; int K; };
    auto side = [&](bool second) __attribute__((always_inline)) {
        const char *A = second ? p2.A2 : g.A, *B = second ? p2.B2 : g.B;
        const int64_t lda = second ? p2.lda2 : g.lda, ldb = second ? p2.ldb2 : g.ldb;
        return Side{A + m0 * lda * 4, B + (B_KC ? n0 * ldb : n0) * 4, lda, ldb, ((reinterpret_cast<uintptr_t>(A) | static_cast<uintptr_t>(lda * 4)) & 15) == 0,
                    ((reinterpret_cast<uintptr_t>(B) | static_cast<uintptr_t>(ldb * 4)) & 15) == 0, static_cast<int>(DUAL && second ? p2.K2 : g.K)};
    };
    const Side s0 = side(other), s1 = side(true);
    // rows and columns beyond the matrices repeat the last one: what they give is never stored
    uint32_t row[TM], col[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) row[i] = static_cast<uint32_t>(M - m0 - 1 < i * 32 + l32 ? M - m0 - 1 : i * 32 + l32);
#pragma unroll
    for (int j = 0; j < TN; ++j) col[j] = static_cast<uint32_t>(g.N - n0 - 1 < j * 32 + l32 ? g.N - n0 - 1 : j * 32 + l32);
    const int steps0 = (s0.K + 15) / 16, steps = steps0 + (DUAL ? (s1.K + 15) / 16 : 0), per = (steps + 7) / 8 * 2;
    const int t_end = steps < (wave + 1) * per ? steps : (wave + 1) * per;
    struct Raw { float a[TM][8], b[TN][8]; };
    // step t: 16 k of 32 that both halves of the wave share in pairs of steps, or the last ones
    auto ask = [&](int t, Raw &r) __attribute__((always_inline)) {
        const bool second = DUAL && t >= steps0;
        const Side &s = DUAL && second ? s1 : s0;
        if (second) t -= steps0;
        const uint32_t lda = static_cast<uint32_t>(s.lda), ldb = static_cast<uint32_t>(s.ldb);
        if (t < s.K / 32 * 2) {
            const int k0 = t / 2 * 32 + (t & 1) * 8;
            const char *a = s.a + k0 * 4, *b = s.b + (B_KC ? static_cast<int64_t>(k0) * 4 : k0 * s.ldb * 4);
            auto along = [&](const char *q, bool vec, float (&x)[8]) __attribute__((always_inline)) {
                if (vec) {
                    const float4 u = reinterpret_cast<const float4 *>(q)[0], v = reinterpret_cast<const float4 *>(q)[1];
                    x[0] = u.x; x[1] = u.y; x[2] = u.z; x[3] = u.w; x[4] = v.x; x[5] = v.y; x[6] = v.z; x[7] = v.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = reinterpret_cast<const float *>(q)[e];
                }
            };
#pragma unroll
            for (int i = 0; i < TM; ++i) along(a + (row[i] * lda + 16u * half) * 4u, s.va, r.a[i]);
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if constexpr (B_KC) {
                    along(b + (col[j] * ldb + 16u * half) * 4u, s.vb, r.b[j]);
                } else {
                    const char *q = b + (16u * half * ldb + col[j]) * 4u;
#pragma unroll
                    for (int e = 0; e < 8; ++e) r.b[j][e] = *reinterpret_cast<const float *>(q + static_cast<int64_t>(e) * s.ldb * 4);
                }
            }
        } else {
            const int k0 = s.K / 32 * 32 + (t - s.K / 32 * 2) * 16 + half * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool in = k0 + e < s.K;
#pragma unroll
                for (int i = 0; i < TM; ++i) r.a[i][e] = in ? *reinterpret_cast<const float *>(s.a + (row[i] * s.lda + k0 + e) * 4) : 0.f;
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    r.b[j][e] = in ? *reinterpret_cast<const float *>(s.b + (B_KC ? col[j] * s.ldb + k0 + e : (k0 + e) * s.ldb + col[j]) * 4) : 0.f;
            }
        }
    };
    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    auto multiply = [&](int t, Raw &r) __attribute__((always_inline)) {
        u32x4 a[TM][3], b[TN][3];
        auto cut = [&](const float (&x)[8], u32x4 (&p)[3]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t u[3];
                split3_pair(x[2 * e], x[2 * e + 1], u);
#pragma unroll
                for (int q = 0; q < 3; ++q) p[q][e] = u[q];
            }
        };
#pragma unroll
        for (int i = 0; i < TM; ++i) cut(r.a[i], a[i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) cut(r.b[j], b[j]);
        if (t + 2 < t_end) ask(t + 2, r);
        constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};       // the six piece products, smallest first
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i][PA[q]]), __builtin_bit_cast(bf16x8, b[j][PB[q]]),
                                                                        acc[i][j], 0, 0, 0);
    };
    {
        Raw x, y;
        int t = wave * per;
        if (t < t_end) ask(t, x);
        if (t + 1 < t_end) ask(t + 1, y);
        for (; t < t_end; t += 2) {
            multiply(t, x);
            if (t + 1 < t_end) multiply(t + 1, y);
        }
    }
    // four columns of rows 16 wave + lane / 16 + 4 p: the epilogue's operands, ahead of the exchange
    char *C = other ? p2.C2 : g.C;
    const int64_t ldc = other ? p2.ldc2 : g.ldc;
    const float *rscale = other ? p2.rscale2 : g.rscale;
    const int c4 = 4 * (lane % 16);
    auto crow = [&](int p) { const int64_t r = m0 + 16 * wave + lane / 16 + 4 * p; return r < M ? r : M - 1; };
    auto ccol = [&](int e) { return n0 + c4 + e < g.N ? n0 + c4 + e : g.N - 1; };
    float e_b[4], e_c[4][4], e_m[4][4], e_s[4];
    if (g.bias)
#pragma unroll
        for (int e = 0; e < 4; ++e) e_b[e] = g.bias[ccol(e)];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if (g.accumulate)
#pragma unroll
            for (int e = 0; e < 4; ++e) e_c[p][e] = reinterpret_cast<const float *>(C)[crow(p) * ldc + ccol(e)];
        if (g.mask)
#pragma unroll
            for (int e = 0; e < 4; ++e) e_m[p][e] = reinterpret_cast<const float *>(g.mask)[crow(p) * g.ldm + ccol(e)];
        if (rscale) e_s[p] = rscale[crow(p)];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) red[wave][i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)][j * 32 + l32] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int lr = 16 * wave + lane / 16 + 4 * p;
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 x = *reinterpret_cast<const float4 *>(&red[w][lr][c4]);
            v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (g.accumulate) v[e] += e_c[p][e];
            if (g.bias) v[e] += e_b[e];
            if (g.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
            if (g.mask) v[e] = e_m[p][e] > 0.f ? v[e] : 0.f;
            if (rscale) v[e] *= e_s[p];
        }
        if (m0 + lr >= M) continue;
        float *out = reinterpret_cast<float *>(C) + (m0 + lr) * ldc + n0 + c4;
        if (n0 + c4 + 4 <= g.N && ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0) {
            *reinterpret_cast<float4 *>(out) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n0 + c4 + e < g.N) out[e] = v[e];
        }
    }
}

// Plain fp32 products of middling size (the 128-row tiles of gemm_split_kernel would not fill the chip): 64 x 64 tiles with
// four waves, a 32 x 32 part each.  Both operands are cut here, the second one as well, which saves the launch that cuts a
// weight matrix beforehand (4-5 us, a third of such a product).  Two LDS buffers and operands fetched two steps ahead: one
// barrier per step and no step waits for memory; three workgroups share a compute unit.
// Also the sum of two products (dual) and two products of one shape (pair), see SmallGemmArgs.

// An operand stored across the reduction index, cut while staged into the same 16-byte units: a thread takes eight k of one
// column (64 neighbouring columns per wave and load).
struct SplitUnitLoader {
    float r[8];
    uint4 pk[3];

    template <bool FULL>
    __device__ __forceinline__ void fetch(const char *base, int64_t ld, int64_t t0, int64_t T, int64_t k0, int64_t k_end, int tid) {
        const int64_t t = t0 + (tid & 63) < T ? t0 + (tid & 63) : T - 1, k = k0 + 8 * (tid >> 6);     // columns beyond T: never stored
        const float *p = reinterpret_cast<const float *>(base) + k * ld + t;
#pragma unroll
        for (int e = 0; e < 8; ++e) r[e] = FULL || k + e < k_end ? p[e * ld] : 0.f;
    }

    __device__ __forceinline__ void cut() {
        uint32_t w[4][3];
#pragma unroll
        for (int e = 0; e < 4; ++e) split3_pair(r[2 * e], r[2 * e + 1], w[e]);
#pragma unroll
        for (int p = 0; p < 3; ++p) pk[p] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
    }

    __device__ __forceinline__ void put(char *s, int tid) const {
#pragma unroll
        for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4 *>(s + Units16<64>::at(p, tid >> 6, tid & 63)) = pk[p];
    }
};

template <bool B_KC>
__global__ __launch_bounds__(256, 3) void gemm_split_mid_kernel(SmallGemmArgs s) {
    constexpr int BT = 64, BYTES = Units16<BT>::BYTES;
    __shared__ __attribute__((aligned(16))) char smem[2][2][BYTES];
    const GemmArgs &g = s.g;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int l32 = lane & 31, half = lane >> 5;
    int bx, by, bz;
    if (!tile_coords(g, &bx, &by, &bz)) return;      // uniform over the workgroup
    const bool second = blockIdx.y != 0;             // pair: the other second operand and result
    const int64_t M = second ? s.M2 : g.M;
    const int64_t m0 = static_cast<int64_t>(by) * BT, n0 = static_cast<int64_t>(bx) * BT;
    if (m0 >= M) return;                             // uniform over the workgroup
    const int nk1 = static_cast<int>((g.K + SBK - 1) / SBK);
    const int nk = nk1 + (s.dual ? static_cast<int>((s.K2 + SBK - 1) / SBK) : 0);

    floatx16 acc[1][1];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[0][0][r] = 0.f;
    SplitRowLoader<BT> la;
    typename std::conditional<B_KC, SplitRowLoader<BT>, SplitUnitLoader>::type lb;
    auto fetch = [&](int t) __attribute__((always_inline)) {
        const bool alt = t >= nk1;                   // uniform over the grid
        const char *A = (alt || second) ? s.A2 : g.A, *B = (alt || second) ? s.B2 : g.B;
        const int64_t lda = (alt || second) ? s.lda2 : g.lda, ldb = (alt || second) ? s.ldb2 : g.ldb;
        const int64_t k0 = static_cast<int64_t>(alt ? t - nk1 : t) * SBK, kend = alt ? s.K2 : g.K;
        if (m0 + BT <= M && k0 + SBK <= kend && g.a_vec) la.fetch_at(A, lda, m0, k0, tid);
        else la.fetch(A, lda, m0, M, k0, kend, g.a_vec, tid);
        if constexpr (B_KC) {
            if (n0 + BT <= g.N && k0 + SBK <= kend && g.b_vec) lb.fetch_at(B, ldb, n0, k0, tid);
            else lb.fetch(B, ldb, n0, g.N, k0, kend, g.b_vec, tid);
        } else {
            if (k0 + SBK <= kend) lb.template fetch<true>(B, ldb, n0, g.N, k0, kend, tid);
            else lb.template fetch<false>(B, ldb, n0, g.N, k0, kend, tid);
        }
    };
    fetch(0);
    la.cut();
    lb.cut();
    la.put(smem[0][0], tid);
    lb.put(smem[0][1], tid);
    if (nk > 1) fetch(1);
    __syncthreads();
    for (int t = 0; t < nk; ++t) {
        const char *As = smem[t & 1][0], *Bs = smem[t & 1][1];
        if (t + 1 < nk) {
            la.cut();
            lb.cut();
            if (t + 2 < nk) fetch(t + 2);
        }
#pragma unroll
        for (int ks = 0; ks < SBK / 16; ++ks) {
            bf16x8 a[3], b[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                a[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(As + Units16<BT>::at(p, 2 * ks + half, wm * 32 + l32)));
                b[p] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(Bs + Units16<BT>::at(p, 2 * ks + half, wn * 32 + l32)));
            }
            // the six piece products, smallest first
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b[0], acc[0][0], 0, 0, 0);
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[2], acc[0][0], 0, 0, 0);
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[1], acc[0][0], 0, 0, 0);
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b[0], acc[0][0], 0, 0, 0);
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[1], acc[0][0], 0, 0, 0);
            acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[0], acc[0][0], 0, 0, 0);
        }
        if (t + 1 < nk) {
            la.put(smem[(t + 1) & 1][0], tid);
            lb.put(smem[(t + 1) & 1][1], tid);
        }
        __syncthreads();
    }
    GemmArgs o = g;
    if (second) { o.C = s.C2; o.ldc = s.ldc2; o.rscale = s.rscale2; o.M = M; }
    store_tile<1, 1>(o, acc, m0 + wm * 32, n0 + wn * 32, l32, half, 0);
}

// Cuts the (small) second operand of a plain product into bf16 pieces laid out in 16-byte units
// Wt[piece][k / 8][n][k % 8], n_pad rows, ku_total units along k, zero beyond N and K.  kc: the source is [n][k]
// (pitch ldw), else [k][n].
// A second source W2 (K2 rows, or columns when kc) follows from k = K1p on.
__global__ __launch_bounds__(256) void split_repack_kernel(const float *W, int64_t ldw, int kc, int64_t K, int64_t N,
                                                           uint16_t *Wt, int64_t n_pad, int64_t ku_total,
                                                           const float *W2 = nullptr, int64_t ldw2 = 0, int64_t K1p = 0,
                                                           int64_t K2 = 0) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t plane = ku_total * n_pad * 8;
    if (t >= plane) return;
    const int64_t ku = t / (n_pad * 8), n = (t / 8) % n_pad, k = 8 * ku + (t % 8);
    float x = (n < N && k < K) ? (kc ? W[n * ldw + k] : W[k * ldw + n]) : 0.f;
    if (W2 && k >= K1p) {
        const int64_t k2 = k - K1p;
        x = (n < N && k2 < K2) ? (kc ? W2[n * ldw2 + k2] : W2[k2 * ldw2 + n]) : 0.f;
    }
    uint32_t p[3];
    split3_pair(x, 0.f, p);
    Wt[t] = static_cast<uint16_t>(p[0]);
    Wt[plane + t] = static_cast<uint16_t>(p[1]);
    Wt[2 * plane + t] = static_cast<uint16_t>(p[2]);
}

// Lays the (small) second operand of a product out as Wt[n][k], k contiguous, rows padded to 16 bytes, for the
// bf16 kernel.  kc: the source already is [n][k] (pitch ldw), else it is [k][n].
__global__ __launch_bounds__(256) void repack_bf16_kernel(const uint16_t *W, int64_t ldw, int kc, int64_t K, int64_t N,
                                                          uint16_t *Wt, int64_t ldt) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t >= N * ldt) return;
    const int64_t n = t / ldt, k = t % ldt;
    Wt[t] = k < K ? (kc ? W[n * ldw + k] : W[k * ldw + n]) : static_cast<uint16_t>(0);
}

// The same operand in the units of gemm_bf16_stream_kernel: Wt[k / 8][n][k % 8], n_pad rows, zero beyond N and K.
__global__ __launch_bounds__(256) void unit_repack_kernel(const uint16_t *W, int64_t ldw, int kc, int64_t K, int64_t N, uint16_t *Wt,
                                                          int64_t n_pad, int64_t ku_total) {
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t >= ku_total * n_pad * 8) return;
    const int64_t ku = t / (n_pad * 8), n = (t / 8) % n_pad, k = 8 * ku + (t % 8);
    Wt[t] = (n < N && k < K) ? (kc ? W[n * ldw + k] : W[k * ldw + n]) : static_cast<uint16_t>(0);
}

// Sums the split partials and applies the epilogue.  A workgroup covers 32 consecutive output elements with 8
// groups of threads; group y adds the partials z = y, y+8, ... in that order, then the 8 group sums are added
// in group order: a fixed summation order, whatever the launch geometry.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmArgs g, int S, const float *part2 = nullptr, char *C2 = nullptr,
                                                          int64_t ldc2 = 0, float *colsum = nullptr) {
    if (blockIdx.y != 0) { g.part = const_cast<float *>(part2); g.C = C2; g.ldc = ldc2; }      // the second problem of a pair
    __shared__ float red[8][32];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int64_t total = g.part ? g.M * g.N : 0;       // (no partials: only the column sums are left to add)
    int64_t t = static_cast<int64_t>(blockIdx.x) * 32 + tx;
    // column sums, in double precision, by the first workgroups: few, and with the longest chains (behind C's, and with a load at a time,
    // they ended the launch by themselves: 256 x 256 of 384 parts 32 us, 128 x 256 of 768 parts 42; 20 without them)
    const int64_t d_blocks = colsum ? (g.N + 31) / 32 : 0;
    if (static_cast<int64_t>(blockIdx.x) < d_blocks) {
        if (blockIdx.y != 0) return;
        __shared__ double dred[8][32];
        double d = 0.0;
        if (t < g.N) {
            int z = ty;
            for (; z + 120 < S; z += 128) {
                float q[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) q[u] = g.colpart[static_cast<int64_t>(z + 8 * u) * g.N + t];
#pragma unroll
                for (int u = 0; u < 16; ++u) d += static_cast<double>(q[u]);
            }
            for (; z < S; z += 8) d += static_cast<double>(g.colpart[static_cast<int64_t>(z) * g.N + t]);
        }
        dred[ty][tx] = d;
        __syncthreads();
        if (ty != 0 || t >= g.N) return;
        d = 0.0;
        for (int y = 0; y < 8; ++y) d += dred[y][tx];
        colsum[t] = static_cast<float>(d);
        return;
    }
    t -= d_blocks * 32;
    float v = 0.f;
    if (t < total) {
        int z = ty;
        for (; z + 56 < S; z += 64) {                   // eight loads on their way, added in order
            float q[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) q[u] = g.part[static_cast<int64_t>(z + 8 * u) * total + t];
#pragma unroll
            for (int u = 0; u < 8; ++u) v += q[u];
        }
        for (; z < S; z += 8) v += g.part[static_cast<int64_t>(z) * total + t];
    }
    red[ty][tx] = v;
    __syncthreads();
    if (ty != 0 || t >= total) return;
    v = 0.f;
    for (int y = 0; y < 8; ++y) v += red[y][tx];
    const int64_t row = t / g.N, col = t % g.N;
    if (g.accumulate) {
        v += g.out_bf16 ? __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t *>(g.C)[row * g.ldc + col]) << 16)
                        : reinterpret_cast<const float *>(g.C)[row * g.ldc + col];
    }
    if (g.bias) v += g.bias[col];
    if (g.relu) v = v > 0.f ? v : 0.f;
    if (g.mask) {
        const float mv = g.mask_bf16 ? __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t *>(g.mask)[row * g.ldm + col]) << 16)
                                     : reinterpret_cast<const float *>(g.mask)[row * g.ldm + col];
        if (!(mv > 0.f)) v = 0.f;
    }
    if (g.rscale) v *= g.rscale[row];
    if (g.out_bf16) reinterpret_cast<uint16_t *>(g.C)[row * g.ldc + col] = static_cast<uint16_t>(f32_to_bf16_rne(v));
    else reinterpret_cast<float *>(g.C)[row * g.ldc + col] = v;
}

// Leaves the sums of gemm_reduce_kernel (and of a pair's second problem) to the end of the epoch; false where it does more than sum.
static bool reduce_later(FinishList *later, const GemmArgs &g, int S, const float *part2, char *C2, int64_t ldc2, float *colsum) {
    if (g.accumulate || g.bias || g.relu || g.mask || g.rscale || g.out_bf16 || (g.part && g.ldc != g.N) || (part2 && ldc2 != g.N) ||
        later->count + 3 > FinishList::MOST)
        return false;
    auto add = [&](FinishTask::Kind kind, const float *part, int64_t n, void *out) {
        FinishTask t{};
        t.kind = kind; t.S = S; t.n = n; t.part = part; t.out = static_cast<float *>(out);
        later->task[later->count++] = t;
    };
    if (g.part) add(FinishTask::SUM, g.part, g.M * g.N, g.C);
    if (part2) add(FinishTask::SUM, part2, g.M * g.N, C2);
    if (colsum) add(FinishTask::COLUMNS, g.colpart, g.N, colsum);
    return true;
}

static int choose_split(int trans_a, int64_t M, int64_t N, int64_t K, int bm, int bn, int bk, bool coarse = false) {
    if (!trans_a) return 1;
    const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    int64_t s = 1536 / (tiles > 0 ? tiles : 1);
    // at least 16 k-steps per split, down to 4 where that leaves compute units without a workgroup (coarse: never)
    int64_t max_by_k = K / (bk * 16);
    if (!coarse && max_by_k * tiles < 256) max_by_k = std::min<int64_t>((256 + tiles - 1) / tiles, K / (bk * 4));
    if (s > max_by_k) s = max_by_k;
    if (s > 1024) s = 1024;
    if (s < 1) s = 1;
    return static_cast<int>(s);
}

static void tile_for(int64_t N, int *bm, int *bn) {
    *bm = 128;
    *bn = (N <= 64) ? 64 : 128;
}

static size_t transposed_b_bytes(int64_t N, int64_t K) {
    return align_up(static_cast<size_t>(N) * ((K + 7) / 8 * 8) * sizeof(uint16_t), 256);
}

// the three bf16 planes of an fp32 weight matrix: rows padded to whole tiles, k to whole steps
static int64_t split_rows(int64_t N) { return (N + 127) / 128 * 128; }
static int64_t split_ld(int64_t K) { return (K + SBK - 1) / SBK * SBK; }
static size_t split_b_bytes(int64_t N, int64_t K) {
    return align_up(static_cast<size_t>(3) * split_rows(N) * split_ld(K) * sizeof(uint16_t), 256);
}

// Units of 16 k that a wave of gemm_bf16_stream_kernel holds, or 0 where it does not apply; its image of the weights
static int stream_units(int64_t K) { return K <= 0 || K > 512 ? 0 : K <= 128 ? 8 : K <= 256 ? 16 : 32; }
static size_t stream_b_bytes(int64_t N, int64_t K) {
    return N > 64 ? static_cast<size_t>(split_rows(N)) * stream_units(K) * 16 * sizeof(uint16_t) : 0;
}

constexpr int64_t NARROW_K = 16384;         // see narrow_product
static size_t narrow_ws_bytes(int64_t M, int64_t N, int64_t K);
static bool small_product(bool bf16, int trans_a, int64_t M, int64_t N, int64_t K, int launches = 1, int trans_b = 0);
static void small_geometry(bool bf16, int trans_a, int64_t M, int64_t N, int64_t K, int *tn, int *S, int64_t *k_chunk);

size_t gemm_ws_bytes(int trans_a, int64_t M, int64_t N, int64_t K) {
    int bm, bn;
    tile_for(N, &bm, &bn);
    // the larger split of the two kernels (they step through K in 16s and 32s)
    const int s = std::max(choose_split(trans_a, M, N, K, bm, bn, BK), choose_split(trans_a, M, N, K, bm, bn, HBK));
    // partial results of every split, and the column sums of B
    size_t b = s > 1 ? align_up(static_cast<size_t>(s) * M * N * sizeof(float), 256) : 0;
    int s_max = s;
    for (const bool bf : {false, true})
        if (trans_a && small_product(bf, trans_a, M, N, K)) {
            int tn, z;
            int64_t chunk;
            small_geometry(bf, trans_a, M, N, K, &tn, &z, &chunk);
            if (z > 1) b = std::max(b, align_up(static_cast<size_t>(z) * M * N * sizeof(float), 256));
            s_max = std::max(s_max, z);
        }
    if (trans_a) b += align_up(static_cast<size_t>(s_max) * N * sizeof(float), 256);
    if (trans_a && N <= 64 && K >= NARROW_K) b = std::max(b, narrow_ws_bytes(M, N, K));
    // room to lay a weight matrix out for the bf16 kernels (bf16 operands) or as its three planes (fp32 operands)
    if (!trans_a) b = std::max({b, transposed_b_bytes(N, K), split_b_bytes(N, K), stream_b_bytes(N, K)});
    return b;
}

size_t gemm_dual_ws_bytes(int64_t N, int64_t K1, int64_t K2) { return split_b_bytes(N, split_ld(K1) + K2); }

constexpr int64_t SPLIT_MIN_MACS = int64_t(1) << 28;     // AUTO: the three-piece form from here on (see split_form)

// Which products take gemm_small_kernel (fp32 ones unless their three-piece form was asked for).  Plain fp32 products, all of those
// that AUTO leaves to the fp32 instruction are candidates (gemm_kernel is the other choice): the launch grows with its 32 x 32
// tiles once they are about four per compute unit, and what it saves, the round trips of a step-by-step reduction, with K.  us
// against gemm_kernel: 10000 x 41 x 16 (626 tiles) 8.4 / 8.1, 4096 x 256 x 16 (1024) 8.6 / 8.7, 10000 x 128 x 16 (1252) 13.7 / 8.9;
// 10000 x 128 x 50 (1252) 14.1 / 14.0, 21557 x 41 x 50 (1348) 13.8 / 11.8; 21557 x 41 x 100 (1348) 14.1 / 14.4, 10000 x 256 x 100
// (2504) 22 / 17; 21557 x 64 x 128 (1348) 13.0 / 13.8, 50000 x 41 x 128 (3126) 25 / 21; 21557 x 41 x 256 17 / 24; 10000 x 41 x
// 602 26 / 54.  A sum of two products replaces two launches of gemm_kernel, so it may have twice the tiles (launches = 2).
// Reductions over vertices (trans_a), whose other kernels stage tiles through LDS step by step: about as far as the small kernel is
// the faster one for every M, with the splits of small_geometry (us small / other, M x N at 2^e multiply-adds, medians over five
// placements of the operands).  fp32, N > 64, up to 2^28.46: 200 x 256 14 / 20 at 2^27, 602 x 256 22 / 26 at 2^28, 100 x 256 23 / 23
// and 602 x 256 26 / 23 at 2^28.4.  fp32, N <= 64 (the other kernel half idle), up to 2^31, where gemm_narrow_kernel does not take them
// (see narrow_product: shorter reductions, little workspace, few rows and very many vertices): 100 x 41 81 / 86 at 2^30, 200 x 41 124 /
// 130, 320 x 64 79 / 81, 602 x 41 118 / 111, 512 x 64 70 / 63 at 2^31, 602 x 41 232 / 197 at 2^32.  bf16, N > 64, up to 2^30.46:
// 200 x 256 21 / 26, 602 x 256 28 / 27, 100 x 100 31 / 33 at 2^30.  bf16, 32 < N <= 64, up to 2^32: 200 x 41 42 / 57, 602 x 64 30 / 32
// at 2^31, 512 x 64 44 / 51, 602 x 41 69 / 64 at 2^32.  bf16, N <= 32, up to 2^30: 100 x 16 60 / 83, 602 x 16 54 / 51 at 2^30, 320 x 16
// 117 / 95 at 2^31.
// Plain bf16 products: from the k on from which its one round trip pays for its loads of W element by element, while its workgroups (32 rows by
// 32 or 64 columns) are few (a sweep of 726 sizes; us, 64 x 64 tiles with the launch that repacks W where they need it / small):
// - taken: 12000 x 32 x 64 5.8 / 5.6, 6000 x 128 x 128 7.3 / 6.5, 3000 x 64 x 256 9.8 / 6.2, 500 x 256 x 602 17.8 / 8.6, 25000 x 16 x 256 10.7 / 9.8;
// - left: 3000 x 128 x 32 6.0 / 6.1, 12000 x 128 x 128 7.8 / 9.7, 25000 x 32 x 64 6.2 / 6.7, and, by the same line, 12000 x 128 x 389 14.4 / 13.4.
// By W^T (both operands along k) the tiles need no repacking: taken 12000 x 16 x 256 8.2 / 7.0, 3000 x 32 x 128 6.3 / 6.4, left 6000 x 64 x 256
// 8.0 / 8.1.  Two products of one shape in one launch replace two of either.
static bool small_product(bool bf16, int trans_a, int64_t M, int64_t N, int64_t K, int launches, int trans_b) {
    if (K <= 0) return false;
    const double macs = static_cast<double>(M) * N * K;
    if (trans_a) return macs <= (bf16 ? (N <= 32 ? 0x1p30 : N <= 64 ? 0x1p32 : 0x1.6p30) : (N <= 64 ? 0x1p31 : 0x1.6p28));
    if (!bf16) return macs < SPLIT_MIN_MACS && ((M + 31) / 32) * ((N + 31) / 32) <= launches * (1024 + 8 * std::max<int64_t>(K - 50, 0));
    const int64_t n_wg = ((M + 31) / 32) * (N <= 32 ? 1 : (N + 63) / 64);
    if (launches > 1) return n_wg <= 400;
    if (trans_b) return N <= 32 && K >= 96 && n_wg <= 400;
    return K >= 64 && n_wg <= (N <= 32 && K >= 96 ? 800 : 400);
}

// Tiles and reduction splits of a small product: N tiles of 64 columns (32 where that is all), and for a reduction over
// vertices splits for the two workgroups that a compute unit holds, each wave with at least one batch.  The tiles of a split run on
// one L2 domain (tile_coords), which holds 64 workgroups, so the splits are dealt in eights, and as many eights are taken as give
// the shortest sweep over two loads of the domains at most (more splits cost more to add up).  512 / tiles splits left one domain
// of a 602-row result with 76 workgroups and another with 57 (us, 602 x 41: fp32 2^31 143 -> 118, bf16 2^30 44 -> 25; 320 x 41 fp32
// 2^31 141 -> 112), and two domains without any where the tiles are more than 64 (bf16 602 x 256 2^30 32 -> 28).
static void small_geometry(bool bf16, int trans_a, int64_t M, int64_t N, int64_t K, int *tn, int *S, int64_t *k_chunk) {
    const int64_t unit = bf16 ? SMALL_UNIT_K<true> : SMALL_UNIT_K<false>, batch = unit * SMALL_UNITS;
    *tn = N <= 32 ? 1 : 2;
    *S = 1;
    const int64_t tiles = ((M + 31) / 32) * ((N + *tn * 32 - 1) / (*tn * 32));
    if (trans_a) {
        constexpr int64_t HELD = 2 * NUM_CU / NUM_XCD;       // workgroups an L2 domain holds
        const int64_t most = K / (4 * batch);                // splits with at least one batch per wave
        auto sweep = [&](int64_t eights) { return static_cast<double>((eights * tiles + HELD - 1) / HELD) / eights; };
        const int64_t e_most = std::min<int64_t>(most / NUM_XCD, std::max<int64_t>(2 * HELD / tiles, 1));
        if (e_most < 1) {
            *S = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(2 * NUM_CU / tiles, most)));
        } else {
            double best = sweep(1);
            for (int64_t e = 2; e <= e_most; ++e) best = std::min(best, sweep(e));
            int64_t e = 1;
            while (sweep(e) > 1.03 * best) ++e;
            *S = static_cast<int>(NUM_XCD * e);
        }
    }
    const int64_t chunk = (K + *S - 1) / *S;
    *k_chunk = (chunk + 4 * unit - 1) / (4 * unit) * (4 * unit);
    *S = static_cast<int>((K + *k_chunk - 1) / *k_chunk);
}

// Which reductions over vertices take gemm_narrow_kernel: those of 16384 vertices and more.  us, gemm_small_kernel (up to 2^31
// multiply-adds) or gemm_kernel -> here: 50 x 41 x 22000 18.5 -> 11.4, 128 x 47 x 60000 27.7 -> 17.9, 256 x 41 x 180000 99 -> 54, 602 x 41 x
// 60000 90 -> 51, 256 x 47 x 306000 164 -> 100 (3.7 TB/s), 602 x 64 x 180000 205 -> 155; below, where few batches leave most of the time
// to the start: 100 x 64 x 9973 12.9 -> 13.2, 128 x 64 x 8192 11.2 -> 14.2, 64 x 7 x 9973 10.0 -> 9.9.  At most 32 rows fill a quarter of its tile: with more than 16 columns that costs it more than the
// loads above 2^18 vertices (32 x 24 x 600000 44 -> 61, 16 x 64 x 600000 65 -> 97; 16 x 64 x 180000 37 -> 35).
static bool narrow_product(int dtype, int mode, int trans_a, int trans_b, int64_t M, int64_t N, int64_t K) {
    return dtype == CAPGNN_F32 && trans_a && !trans_b && N <= 64 && mode != CAPGNN_F32_PRODUCT_SPLIT && K >= NARROW_K &&
           !(M <= 32 && N > 16 && K > (1 << 18));
}

// Its splits: as many as make one workgroup per compute unit, or two where a split is longer than 1024 vertices, in eights.  Between the
// two some compute units have twice the work of others (256 x 64 x 40000 with 256 workgroups 23.5 us, 320 33.4, 512 27.2), and
// the more splits the more parts to add up.
static int narrow_splits(int64_t M, int64_t K) {
    const int64_t gy = (M + 127) / 128, s = (gy * K > (int64_t(1) << 18) ? 2 : 1) * NUM_CU / gy;
    return static_cast<int>(std::max<int64_t>(s > 8 ? s / 8 * 8 : s, 1));
}

static size_t narrow_ws_bytes(int64_t M, int64_t N, int64_t K) {
    const size_t s = static_cast<size_t>(narrow_splits(M, K));
    return align_up(s * M * N * sizeof(float), 256) + align_up(s * N * sizeof(float), 256);
}

// AUTO: smaller products stay on the fp32 instruction (the caller is told the limit), and so do weight gradients at most 64
// columns wide (half of the threads that stage their operands would idle; measured slower)
static bool split_form(int mode, int trans_a, int64_t M, int64_t N, int64_t K) {
    if (mode != CAPGNN_F32_PRODUCT_AUTO) return mode == CAPGNN_F32_PRODUCT_SPLIT;
    return M * N >= SPLIT_MIN_MACS / (K > 0 ? K : 1) && !(trans_a && N <= 64);
}

// the sum of two products: a layer's forward products count as one, those of its input gradient each for itself
static bool split_sum(int mode, int trans_b, int64_t M, int64_t N, int64_t K1, int64_t K2) {
    if (trans_b) return split_form(mode, 0, M, N, K1) && split_form(mode, 0, M, N, K2);
    return split_form(mode, 0, M, N, K1 + K2);
}

// tiles 64 columns wide keep four waves; 128-column tiles run eight
static void launch_split_tiles(const GemmArgs &g, int bn, dim3 grid, const uint16_t *Wt, int64_t ku_total, int64_t n_pad, hipStream_t st) {
    if (bn == 64) hipLaunchKernelGGL((gemm_split_kernel<128, 64>), grid, dim3(256), 0, st, g, Wt, ku_total, n_pad);
    else hipLaunchKernelGGL((gemm_split_kernel<128, 128, 8>), grid, dim3(512), 0, st, g, Wt, ku_total, n_pad);
}

// gemm_split_cols_kernel: column tiles of 32 in a workgroup's tile, reduction splits (workgroups per tile), parts of each, vertices of a
// wave in a part.  At most `most` partial results.  A step of 16 vertices takes a wave 2.4 us with 128 columns and 1.45 us with 64, a
// workgroup's start and end 11 and 8 us (256 x 256 by 40000 and 306000, 100 x 256 by 70001 and 306000), a compute unit holds one workgroup,
// and the tiles of a split share an L2 domain, so the splits come in eights where they are that many.  So 128 columns but for short
// reductions and for columns that fill half of the last tile: us with the better splits, 128 and 64 columns: 256 x 256 x 306000 189, 218;
// 602 x 200 x 30000 57, 65; 256 x 256 x 40000 36.0, 35.5; 128 x 128 x 100000 30.1, 27.5; 97 x 131 x 50001 29.5, 25.4.
struct ColsPlan { int tb, S, parts; int64_t chunk; };
static ColsPlan cols_plan(bool bf16, int64_t M, int64_t N, int64_t K, int most, int products = 1) {
    const int64_t unit = bf16 ? 64 : 32;                // vertices of a wave are whole turns of its loop
    ColsPlan best{4, 1, 1, 0};
    double best_us = 1e30;
    for (int tb : {4, 2}) {
        const int64_t tiles = products * ((M + 127) / 128) * ((N + tb * 32 - 1) / (tb * 32)), held = NUM_CU / NUM_XCD;
        const double step = bf16 ? (tb == 4 ? 0.8 : 0.6) : tb == 4 ? 2.4 : 1.45, ends = bf16 ? (tb == 4 ? 9.0 : 7.0) : tb == 4 ? 11.0 : 8.0;
        for (int S = 1; S <= most && S <= 2 * NUM_CU; S += S < 8 ? 1 : 8) {
            const int64_t per_domain = S < NUM_XCD ? (S * tiles + NUM_XCD - 1) / NUM_XCD : S / NUM_XCD * tiles, steps = (K + 64 * S - 1) / (64 * S);
            const double us = (per_domain + held - 1) / held * (steps * step + ends) + (S > 1 ? 1.6e-6 * products * S * M * N : 0.0);
            if (us < best_us) {
                best_us = us;
                best.tb = tb;
                best.S = S;
            }
        }
    }
    const int64_t wave = (K + 4 * best.S - 1) / (4 * best.S);
    best.parts = static_cast<int>(std::max<int64_t>(std::min<int64_t>((wave + COLS_CHAIN - 1) / COLS_CHAIN, (most + 4 * best.S - 1) / (4 * best.S)), 1));
    best.chunk = ((wave + best.parts - 1) / best.parts + unit - 1) / unit * unit;
    return best;
}

// Which of gemm_small_kernel's bf16 reductions over vertices gemm_bf16_cols_kernel takes (it takes all of those that the small kernel leaves): its
// ends cost 9 us, its tiles are 128 rows high, and it reads faster.  From a sweep of both (550 sizes, M 16 to 602, N 2 to 256, K 1000 to 250000: 0.89
// of the small kernel's time with the faster one each time), us small -> here, M x N x K:
// - N <= 64, from 6 M elements of X: 389 x 16 x 20000 20.4 -> 13.8, 100 x 41 x 100000 20.3 -> 17.7; below that little is left (128 x 32 x 40000
//   15.5, here 15.0; 100 x 16 x 40000 14.6, 14.4), and not for X that fills less than three quarters of a tile: 50 x 41 x 250000 18.6, here 20.9,
//   16 x 64 x 250000 17.2, 18.6;
// - N <= 128, from 2^21 elements over 16384 vertices and 2^22 below: 128 x 100 x 20000 15.4 -> 14.6; left are 389 x 100 x 10000 16.9, here 16.6,
//   200 x 128 x 10000 14.6, 15.3, and, with few columns of X, 16 x 100 x 250000 19.4, 24.5, 50 x 121 x 200000 28, 31;
// - above, from 2^20 and 2^21 elements, left 50 x 256 x 20000 15.3, here 14.8, 200 x 256 x 10000 17.3, 17.3, 200 x 200 x 5000 13.8, 14.8, 1000 x 600
//   x 2000 24.5, 26.1; and whenever X has 512 columns and more with N <= 256 (the small kernel's tiles fill the chip more than once):
//   602 x 256 x 1000 22.1 -> 15.5.
static bool bf16_cols_pays(int64_t M, int64_t N, int64_t K) {
    const int64_t x = M * K;
    if (N <= 64) return M >= 96 && x >= 6000000;
    if (M <= 32 || (M < 64 && N <= 128 && K >= (1 << 17))) return false;
    if (N > 128 && N <= 256 && M >= 512) return true;
    return x >= (int64_t(1) << (20 + (N <= 128) + (K < 16384)));
}

// Which three-piece products of middling size gemm_split_quarters_kernel takes: those whose 64 x 64 tiles are two per compute unit at most, or three
// with a long reduction; by W^T, whose rows it reads in 16-byte pieces, fewer.  us, gemm_split_mid_kernel -> here, M x N x K (280 sizes): 4096 x 256 x 602 27.4 ->
// 17.0, 8820 x 64 x 602 28.3 -> 15.5, 15000 x 128 x 256 17.1 -> 15.0, 21557 x 64 x 256 17.7 -> 14.1, 30000 x 64 x 389 25.9 -> 22.4, 8820 x 256 x 389 28.7 -> 26.6, 21557 x 128 x 256 21.0 ->
// 19.8; not 21557 x 128 x 128 14.0, here 13.9, nor 15000 x 256 x 256 18.9, 24.1.  By W^T: 4096 x 256 x 256 17.0 -> 13.8, 21557 x 64 x 200 20.0 -> 17.7; not 8820 x 128 x
// 256 19.6, here 21.3, nor 21557 x 128 x 128 17.8, 20.8.
static bool quarters_pay(int64_t M, int64_t N, int64_t K, int trans_b) {
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
    if (trans_b) return tiles <= 256 || (tiles <= 480 && K <= 224);
    return tiles <= 512 || (tiles <= 768 && K >= 256);
}

static void launch_cols(const SmallGemmArgs &s, bool bf16, const ColsPlan &p, dim3 grid, hipStream_t st) {
#define CG_COLS(TB_, SUMS_) if (p.tb == TB_ && !!s.g.colpart == SUMS_) { \
        if (bf16) hipLaunchKernelGGL((gemm_bf16_cols_kernel<TB_, SUMS_>), grid, dim3(256), 0, st, s, p.parts); \
        else hipLaunchKernelGGL((gemm_split_cols_kernel<TB_, SUMS_>), grid, dim3(256), 0, st, s, p.parts); }
    CG_COLS(4, false) CG_COLS(4, true) CG_COLS(2, false) CG_COLS(2, true)
#undef CG_COLS
}

// what 32-bit offsets of 16 rows and row numbers reach
static bool cols_reach(int64_t K, int64_t lda, int64_t ldb) { return K < (int64_t(1) << 30) && lda < (1 << 24) && ldb < (1 << 24); }

// workgroups of one product: tiles times splits, padded to whole rounds of the L2 domains where the splits are dealt to them
static int64_t cols_grid(const ColsPlan &p, int64_t M, int64_t N) {
    const int64_t tiles = (M + 127) / 128 * ((N + p.tb * 32 - 1) / (p.tb * 32));
    return p.S < NUM_XCD ? p.S * tiles : (p.S + NUM_XCD - 1) / NUM_XCD * NUM_XCD * tiles;
}

template <int NS, int KH>
static void launch_split_stream_cfg(const GemmArgs &g, const uint16_t *Wt, uint32_t ku_total, uint32_t n_pad, hipStream_t st) {
    const int64_t gy = (g.N + NS / KH * 32 - 1) / (NS / KH * 32);
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>((g.M + 31) / 32, NUM_CU * split_stream_held(NS, KH) / gy)), static_cast<unsigned>(gy)), block(NS * 64);
#define CG_FORM(D_, M_) if (!!g.A2 == D_ && !!g.mask == M_) \
        hipLaunchKernelGGL((gemm_split_stream_kernel<NS, KH, D_, M_>), grid, block, 0, st, g, Wt, ku_total, n_pad);
    CG_FORM(false, false) CG_FORM(false, true) CG_FORM(true, false) CG_FORM(true, true)
#undef CG_FORM
}

// Which products of more than 64 columns (306 k x 47 x 256 125 us there, 99 in 64-column tiles) gemm_split_stream_kernel takes; M rows in
// all, K: both operands of a sum, the first padded to whole steps.  Its time goes by 128 and 256 k, that of gemm_split_kernel by steps of 32
// and by full rounds of its tiles over the chip.  us alone, gemm_split_kernel -> here, M x N x K:
// - up to 32 k without a mask it is level or slower: 306000 x 128 x 16 44 -> 53 (masked x 32 100 -> 78); from there to 128 k 0.65 to 1 of
//   the time: 306000 x 128 x 40 62 -> 55, x 128 94 -> 75, x 256 x 128 174 -> 116, 26000 x 128 x 128 15.2 -> 13.5;
// - 129 to 192 k it multiplies zeros as well: 306000 x 128 x 160 106 -> 120, x 132 x 160 161 -> 202, x 256 x 192 213 -> 226; so only where the tiles'
//   last round leaves more than a quarter of their time idle: 20000 x 200 x 192 25.2 -> 21.6, 33000 x 256 x 160 36 -> 36, masked 70000 x 100 x 192 46 -> 34;
// - above, 0.8 to 1: 306000 x 256 x 256 265 -> 238 (masked 361 -> 245), x 200 248 -> 237; but as before for the seven whole steps of 224 k (130000 x 160 x 224
//   1.08, masked less), and for one incomplete round of 128 columns (26000 x 68 x 256 1.04, x 96 x 192 1.09);
// - columns that are no whole groups of four cost it a second pass over them: 306000 x 66 x 160 95 -> 139, x 121 x 160 0.75 as fast; it still
//   gains where the tiles leave time idle, most of its waves' 32 columns are there and few k are zero: 70000 x 121 x 100 33 -> 29, masked 42 -> 32.
static bool split_stream_pays(int64_t M, int64_t N, int64_t K, bool masked) {
    if (N <= 64 || N > 256 || K > 256 || M < 12288) return false;
    const int64_t tiles = (M + 127) / 128 * ((N + 127) / 128);
    const bool idle = tiles * 4 <= (tiles + NUM_CU - 1) / NUM_CU * NUM_CU * 3;
    if (N % 4 != 0) return idle && N % 32 > 16 && K >= 96 && K <= 128;
    if (K <= 128) return K > 32 || masked;
    if (K <= 192 || (K == 224 && !masked)) return idle;
    return tiles > NUM_CU || N > 128 || idle;
}

// weights cut into Wt; false where its rows do not start on 16 bytes, or it does not pay
static bool launch_split_stream(const GemmArgs &g, const uint16_t *Wt, int64_t ku_total, int64_t n_pad, hipStream_t st) {
    const bool rows16 = g.a_vec && aligned16(g.A) && aligned16(g.C) && g.ldc % 4 == 0 && (!g.mask || (aligned16(g.mask) && g.ldm % 4 == 0)) &&
                        (!g.A2 || (aligned16(g.A2) && g.lda2 % 4 == 0));
    if (!rows16 || g.accumulate || g.part || g.out_bf16 || !split_stream_pays(g.M, g.N, g.K, g.mask != nullptr) ||
        g.lda >= (1 << 22) || g.lda2 >= (1 << 22) || g.ldc >= (1 << 22) || g.ldm >= (1 << 22))
        return false;
    const uint32_t ku = static_cast<uint32_t>(ku_total), np = static_cast<uint32_t>(n_pad);
    if (g.K > 128) launch_split_stream_cfg<8, 2>(g, Wt, ku, np, st);
    else if (g.N > 128) launch_split_stream_cfg<8, 1>(g, Wt, ku, np, st);
    else launch_split_stream_cfg<4, 1>(g, Wt, ku, np, st);
    return true;
}

template <bool BF16, bool A_KC, bool B_KC>
static void launch_tiles(const GemmArgs &g, int bn, dim3 grid, hipStream_t st) {
    if (bn == 64) hipLaunchKernelGGL((gemm_kernel<BF16, A_KC, B_KC, 128, 64>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gemm_kernel<BF16, A_KC, B_KC, 128, 128>), grid, dim3(256), 0, st, g);
}

// bm64: tiles of 64 rows (plain products only)
template <bool A_KC, bool B_KC>
static void launch_bf16_tiles(const GemmArgs &g, int bn, bool bm64, dim3 grid, hipStream_t st) {
    if constexpr (A_KC) {
        if (bm64) {
            hipLaunchKernelGGL((gemm_bf16_kernel<A_KC, B_KC, 64, 64>), grid, dim3(256), 0, st, g);
            return;
        }
    }
    if (bn == 64) hipLaunchKernelGGL((gemm_bf16_kernel<A_KC, B_KC, 128, 64>), grid, dim3(256), 0, st, g);
    else hipLaunchKernelGGL((gemm_bf16_kernel<A_KC, B_KC, 128, 128>), grid, dim3(256), 0, st, g);
}

// Which products of more than 64 columns (980 k x 47 x 128 104 us there, 91 in tiles; x 256 146 / 149) gemm_bf16_stream_kernel takes: from how
// many rows on, or a negative number where never.  Its time goes by 128, 256 and 512 k and by 128 columns (up to there) or 256; the tiles
// (64 rows while they are few) waste less of both, and need no load of weights per workgroup, but read rows that end inside eight k
// element by element.  So it depends on the reduction (up to 64, 128, 256, below 400 and up to 512; whole eights or not), on whether three
// quarters of its columns are there, on the mask, which the tiles read as well as it does, and, above 128 columns, on the size of the result
// rather than on its rows.  Columns that are no whole eights cost it a second pass over them.  A sweep of both kernels (17600 sizes, 16 k to
// 980 k rows, 66 to 1000 columns, 6 to 512 k) took 0.81 of the tiles' time by these lines, 0.86 with it wherever it applies and 0.81 with the
// faster one each time.  us, tiles -> here, rows x columns x k:
//   at most 128 columns: 16384 x 72 x 64 6.2 -> 6.6, 25000 x 96 x 64 0.91; 16384 x 128 x 128 0.86; 100000 x 72 x 264 28 -> 36; 100000 x 128 x 448 0.93
//   masked: 33000 x 72 x 32 1.11, 50000 x 72 x 32 1.02; 33000 x 128 x 128 0.88; 100000 x 96 x 400 36 -> 39
//   full: 16384 x 256 x 256 12.6 -> 10.7, 980000 x 256 x 256 322 -> 195; masked 25000 x 256 x 256 1.15, 66000 x 256 x 256 0.9, 16384 x 512 x 128 0.75
//   not full: 16384 x 160 x 160 1.18, 33000 x 160 x 160 0.97; masked 50000 x 320 x 160 26 -> 31, 100000 x 160 x 160 0.64
//   ragged: 100000 x 66 x 320 1.64, 50000 x 300 x 32 1.35, masked 50000 x 300 x 8 2.1; but 33000 x 250 x 100 0.69, 100000 x 132 x 128 38 -> 26
static int64_t bf16_stream_rows(int64_t N, int64_t K, bool masked) {
    constexpr int64_t Mi = int64_t(1) << 20;
    if (N <= 64 || !stream_units(K)) return -1;
    const bool wide = N > 128, full = 3 * ((N + 255) / 256 * 256) < 4 * N, odd = K % 8 != 0;
    const int band = K <= 64 ? 0 : K <= 128 ? 1 : K <= 256 ? 2 : K < 400 ? 3 : 4;
    if (!wide) {
        if (band == 3) return -1;
        if (N % 8 != 0) return masked || !odd || band == 4 ? -1 : band == 2 ? 49152 : 24576;
        if (masked) return band == 4 ? 65536 : band == 1 || (band == 2 && !odd) ? 24576 : 49152;
        return band == 4 && odd ? 49152 : band == 0 || (band == 2 && odd) ? 24576 : 16384;
    }
    int64_t result;                     // elements
    if (N % 8 != 0) {
        if (masked || (!odd && (band == 0 || band == 3))) return -1;
        if (full) result = band == 1 || band == 4 || (odd && band != 3) ? 0 : 8 * Mi;
        else result = band == 4 || (odd && (band == 1 || band == 2)) ? 4 * Mi : band == 3 ? 8 * Mi : 12 * Mi;
    } else if (!masked) {
        result = full || band == 1 || band == 4 ? 0 : 4 * Mi;
    } else if (band == 1 || band == 4 || (odd && band == 0)) {
        result = full ? 0 : 4 * Mi;
    } else {
        result = odd ? 8 * Mi : full && band != 2 ? 7 * Mi : band == 0 ? 12 * Mi : 13 * Mi;
    }
    return std::max<int64_t>(16384, (result + N - 1) / N);
}

static bool bf16_stream_pays(int64_t M, int64_t N, int64_t K, bool masked) {
    const int64_t rows = bf16_stream_rows(N, K, masked);
    return rows > 0 && M >= rows;
}

template <int KS, int NS>
static void launch_stream_cfg(const GemmArgs &g, const uint16_t *Wt, uint32_t n_pad, hipStream_t st) {
    constexpr int HELD = NUM_CU * stream_held(KS, NS);
    const int64_t tiles = (g.M + 31) / 32, gy = (g.N + NS * 32 - 1) / (NS * 32);
    const dim3 grid(static_cast<unsigned>(std::min<int64_t>(tiles, std::max<int64_t>(HELD / gy, 1))), static_cast<unsigned>(gy));
    if (g.mask) hipLaunchKernelGGL((gemm_bf16_stream_kernel<KS, NS, true>), grid, dim3(NS * 64), 0, st, g, Wt, n_pad);
    else hipLaunchKernelGGL((gemm_bf16_stream_kernel<KS, NS, false>), grid, dim3(NS * 64), 0, st, g, Wt, n_pad);
}

static void launch_stream(const GemmArgs &g, const uint16_t *Wt, uint32_t n_pad, hipStream_t st) {
    const int ks = stream_units(g.K);
#define CG_STREAM(KS_) if (ks == KS_) { if (g.N <= 128) launch_stream_cfg<KS_, 4>(g, Wt, n_pad, st); \
        else launch_stream_cfg<KS_, 8>(g, Wt, n_pad, st); }
    CG_STREAM(8) CG_STREAM(16) CG_STREAM(32)
#undef CG_STREAM
}

// Epilogue operands held through the loop cost A W of at most 32 columns one of four waves per SIMD, and A W^T of more than 32 one of three:
// worth it while the workgroups that are left are all there are (A W: 15000 x 32 x 200, 469 workgroups, 9.0 us held, 9.5 not; masked A W^T:
// 4096 x 256 x 112 10.6 held, 11.5 not), not where one more per compute unit holds the rest of them (30000 x 20 x 8, 938, 8.5 held, 6.4 not;
// 10000 x 128 x 100 by W^T, 626, 16.0 held, 12.5 not; with more workgroups or k that one holds again: 7000 x 200 x 128, 876 of them, 15.1
// held, 15.9 not; 20000 x 41 x 300 24.8, 28.3).
// bf16 reductions of at most 32 columns: registers for two waves per SIMD while X is small and its workgroups are more than the compute units
// or their chains long (us, one wave and two: 200 x 32 x 12000 16.5, 12.3; 602 x 5 x 5000 15.3, 11.1; 16 x 32 x 66000 17.1, 11.1; equal at
// 512 x 32 x 5000), one beyond (602 x 32 x 30000 24.5, 46.2; 602 x 5 x 150000 92, 294) and where a few workgroups make short chains (in a
// layer, with column sums, 128 x 31 x 1469 7.5, 11.4).
static void launch_small(const SmallGemmArgs &s, bool bf16, bool akc, bool bkc, int tn, dim3 grid, hipStream_t st) {
#define CG_SMALL_CASE(BF, AK, BK_, TN_, HOLD_)                                                                                 \
    if (bf16 == BF && akc == AK && bkc == BK_ && tn == TN_)                                                                    \
        hipLaunchKernelGGL((gemm_small_kernel<BF, AK, BK_, TN_, HOLD_>), grid, dim3(256), 0, st, s);
    CG_SMALL_CASE(false, true, false, 2, true) CG_SMALL_CASE(false, true, true, 1, true)
    const int64_t n_wg = static_cast<int64_t>(grid.x) * grid.y;
    if (n_wg > 3 * NUM_CU) {
        CG_SMALL_CASE(false, true, false, 1, false)
    } else {
        CG_SMALL_CASE(false, true, false, 1, true)
    }
    if (n_wg > 2 * NUM_CU && n_wg <= 3 * NUM_CU && s.g.K + (s.dual ? s.K2 : 0) <= 256) {
        CG_SMALL_CASE(false, true, true, 2, false)
    } else {
        CG_SMALL_CASE(false, true, true, 2, true)
    }
    CG_SMALL_CASE(false, false, false, 1, false) CG_SMALL_CASE(false, false, false, 2, false)
    CG_SMALL_CASE(false, false, true, 1, false) CG_SMALL_CASE(false, false, true, 2, false)
    if (s.g.M * s.g.K * grid.y <= (int64_t(1) << 23) && (n_wg > NUM_CU || s.g.K >= (1 << 14))) {
        CG_SMALL_CASE(true, false, false, 1, true)
    } else {
        CG_SMALL_CASE(true, false, false, 1, false)
    }
    CG_SMALL_CASE(true, false, false, 2, false)
    CG_SMALL_CASE(true, true, false, 1, true) CG_SMALL_CASE(true, true, false, 2, true)
    CG_SMALL_CASE(true, true, true, 1, true) CG_SMALL_CASE(true, true, true, 2, true)
    CG_SMALL_CASE(true, false, true, 1, false) CG_SMALL_CASE(true, false, true, 2, false)
#undef CG_SMALL_CASE
}

// Products of a layer's backward pass that wait for one launch (see gemm_small_batch_kernel)
struct SmallBatch {
    SmallBatchArgs args{};
    dim3 grid[3];
    bool bf16 = false;
    int count = 0, tw = 0, tx = 0;
};

// Takes a product where it fits: weight gradients of one width and one input gradient, each with what the chip holds of workgroups at most, and
// short reductions (bf16 ones of at most 32 columns only where the form for two waves per SIMD is due, see launch_small)
static bool batch_small(SmallBatch *b, const SmallGemmArgs &s, bool bf16, bool akc, bool bkc, int tn, dim3 grid) {
    if (!b || b->count == 3 || akc != bkc || (b->count && b->bf16 != bf16) || static_cast<int64_t>(grid.x) * grid.y > 2 * NUM_CU) return false;
    if (akc ? b->tx != 0 : (b->tw != 0 && b->tw != tn) || s.g.K > 32768 ||
                           (bf16 && tn == 1 && !(s.g.M * s.g.K * grid.y <= (int64_t(1) << 23) && (static_cast<int64_t>(grid.x) * grid.y > NUM_CU || s.g.K >= (1 << 14)))))
        return false;
    const int i = b->count++;
    b->bf16 = bf16;
    (akc ? b->tx : b->tw) = tn;
    b->args.task[i] = s;
    b->args.nx[i] = static_cast<int>(grid.x);
    b->args.plain[i] = akc;
    b->grid[i] = grid;
    return true;
}

int launch_small_batch(SmallBatch *b, hipStream_t st) {
    if (b->count == 1) {
        launch_small(b->args.task[0], b->bf16, b->args.plain[0], b->args.plain[0], b->args.plain[0] ? b->tx : b->tw, b->grid[0], st);
    } else if (b->count > 1) {
        int at = 0;
        for (int i = 0; i < 3; ++i) {
            b->args.first[i] = at;
            if (i < b->count) at += static_cast<int>(b->grid[i].x * b->grid[i].y);
        }
        b->args.first[3] = at;
        const int tw = std::max(b->tw, 1), tx = std::max(b->tx, 1);
#define CG_BATCH(BF_, TW_, TX_) if (b->bf16 == BF_ && tw == TW_ && tx == TX_) \
        hipLaunchKernelGGL((gemm_small_batch_kernel<BF_, TW_, TX_>), dim3(static_cast<unsigned>(at)), dim3(256), 0, st, b->args);
        CG_BATCH(false, 1, 1) CG_BATCH(false, 1, 2) CG_BATCH(false, 2, 1) CG_BATCH(false, 2, 2)
        CG_BATCH(true, 1, 1) CG_BATCH(true, 1, 2) CG_BATCH(true, 2, 1) CG_BATCH(true, 2, 2)
#undef CG_BATCH
    }
    b->count = b->tw = b->tx = 0;
    CG_HIP(hipGetLastError());
    return CAPGNN_OK;
}

// the calling thread's, empty
SmallBatch *small_batch_begin() {
    thread_local SmallBatch b;
    b.count = b.tw = b.tx = 0;
    return &b;
}

static void launch_narrow(const SmallGemmArgs &s, dim3 grid, hipStream_t st) {
    if (s.g.N <= 16) hipLaunchKernelGGL(gemm_narrow_kernel<1>, grid, dim3(256), 0, st, s);
    else if (s.g.N <= 32) hipLaunchKernelGGL(gemm_narrow_kernel<2>, grid, dim3(256), 0, st, s);
    else if (s.g.N <= 48) hipLaunchKernelGGL(gemm_narrow_kernel<3>, grid, dim3(256), 0, st, s);
    else hipLaunchKernelGGL(gemm_narrow_kernel<4>, grid, dim3(256), 0, st, s);
}

static void launch_quarters(const SmallGemmArgs &s, bool bkc, dim3 grid, hipStream_t st) {
    if (bkc && s.dual) hipLaunchKernelGGL((gemm_split_quarters_kernel<true, true>), grid, dim3(256), 0, st, s);
    else if (bkc) hipLaunchKernelGGL((gemm_split_quarters_kernel<true, false>), grid, dim3(256), 0, st, s);
    else if (s.dual) hipLaunchKernelGGL((gemm_split_quarters_kernel<false, true>), grid, dim3(256), 0, st, s);
    else hipLaunchKernelGGL((gemm_split_quarters_kernel<false, false>), grid, dim3(256), 0, st, s);
}

int launch_gemm(int trans_a, int trans_b, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
                const void *B, int64_t ldb, void *C, int64_t ldc, int dtype, int out_f32, int accumulate,
                const float *bias, int relu, const void *relu_mask, int64_t ldm, void *ws, size_t ws_bytes,
                hipStream_t stream, const float *row_scale, int f32_product, float *colsum, FinishList *later, SmallBatch *batch) {
    if (colsum && (!trans_a || trans_b)) CG_FAIL(CAPGNN_EINVAL, "gemm: column sums are formed by X^T G alone");
    if (dtype != CAPGNN_F32 && dtype != CAPGNN_BF16) CG_FAIL(CAPGNN_EINVAL, "gemm: unknown dtype %d", dtype);
    if (f32_product != CAPGNN_F32_PRODUCT_AUTO && f32_product != CAPGNN_F32_PRODUCT_NATIVE && f32_product != CAPGNN_F32_PRODUCT_SPLIT)
        CG_FAIL(CAPGNN_EINVAL, "gemm: unknown form of the fp32 product %d", f32_product);
    if (M < 0 || N < 0 || K < 0) CG_FAIL(CAPGNN_EINVAL, "gemm: negative size");
    if (M == 0 || N == 0) return CAPGNN_OK;
    if (!A || !B || !C) CG_FAIL(CAPGNN_EINVAL, "gemm: NULL operand");
    if (lda < (trans_a ? M : K) || ldb < (trans_b ? K : N) || ldc < N || (relu_mask && ldm < N))
        CG_FAIL(CAPGNN_EINVAL, "gemm: leading dimension too small");
    if (M >= (int64_t(1) << 31) * 64 || N > (1 << 22)) CG_FAIL(CAPGNN_EINVAL, "gemm: size out of range");
    const int es = elem_bytes(dtype);
    int bm, bn;
    tile_for(N, &bm, &bn);
    const int64_t tiles128 = ((M + 127) / 128) * ((N + 127) / 128), tiles64 = ((M + 63) / 64) * ((N + 63) / 64);
    // bf16 operands whose rows start on 16-byte boundaries run on the bf16 matrix cores, in 64 x 64 tiles while tiles of
    // 128 rows are few (20000 x 256 x 256: 17.5 -> 15.5 us; 306000 x 256 x 256: 133 against 111).  The second operand of a
    // product with a plain first operand is a weight matrix, repacked into the workspace first unless it is stored along
    // the reduction index already, or the product so short that the repacking launch is a good part of it (21557 x 128 x 50:
    // 8.9 -> 7.2 us; 5000 x 256 x 602: 18.6 against 16.6)
    const bool b_aligned = aligned16(B) && (ldb * 2) % 16 == 0;
    const bool repack_b = dtype == CAPGNN_BF16 && !trans_a && ws && ws_bytes >= transposed_b_bytes(N, K) &&
                          !(b_aligned && (trans_b || (tiles64 <= 768 && K <= 256)));
    // An empty reduction, which leaves the epilogue of zeros, is gemm_kernel's: it does no step and reads neither operand.
    const bool half_path = dtype == CAPGNN_BF16 && K > 0 && aligned16(A) && (lda * 2) % 16 == 0 && (repack_b || b_aligned) &&
                           (!trans_a || trans_b || cols_reach(K, lda, ldb));
    // fp32 operands as three bf16 pieces each (see gemm_split_kernel)
    const int mode = f32_product;
    const bool split_path = dtype == CAPGNN_F32 && K > 0 && !(trans_a && trans_b) && split_form(mode, trans_a, M, N, K) &&
                            (trans_a ? cols_reach(K, lda, ldb) : ws && ws_bytes >= split_b_bytes(N, K));
    // gemm_split_mid_kernel while its tiles fit the chip at once (three workgroups per compute unit)
    const bool mid_reach = split_path && !trans_a && K < (1 << 30) && lda < (1 << 22) && ldb < (1 << 22);
    const bool mid = mid_reach && tiles64 <= 768, quarters = mid && quarters_pay(M, N, K, trans_b);
    const bool half_cols = half_path && trans_a && !trans_b;
    bool small_path = small_product(dtype == CAPGNN_BF16, trans_a, M, N, K, 1, trans_b) && !(split_path && mode == CAPGNN_F32_PRODUCT_SPLIT);
    if (half_cols && small_path && bf16_cols_pays(M, N, K)) {
        // (with too little room for the parts of these splits, there may be enough for the fewer of the small kernel)
        const size_t s = choose_split(trans_a, M, N, K, bm, bn, HBK), parts = s > 1 ? s * M * N * sizeof(float) : 0;
        const size_t need = colsum ? align_up(parts, 256) + s * N * sizeof(float) : parts;
        small_path = need > 0 && (!ws || ws_bytes < need);
    }
    const int bk = (half_path || split_path) ? HBK : BK;
    static_assert(SBK == HBK, "the two bf16 kernels step through K alike");
    int S = choose_split(trans_a, M, N, K, bm, bn, bk), tn = 0;
    int64_t small_chunk = 0;
    if (small_path) small_geometry(dtype == CAPGNN_BF16, trans_a, M, N, K, &tn, &S, &small_chunk);
    if (S > 1 && (!ws || ws_bytes < static_cast<size_t>(S) * M * N * sizeof(float))) {
        // too little room for that many splits: a reduction of few steps needs none at all on the tiled kernels
        small_path = false;
        S = choose_split(trans_a, M, N, K, bm, bn, bk, true);
    }
    const bool narrow = narrow_product(dtype, mode, trans_a, trans_b, M, N, K) && ws && ws_bytes >= narrow_ws_bytes(M, N, K);
    if (narrow) {
        small_path = false;
        S = narrow_splits(M, K);
        bn = 64;
    }
    if (small_path) {
        bm = 32;
        bn = 32 * tn;
    }
    const bool mid_path = !small_path && mid, cols_path = trans_a && !trans_b && (split_path || half_cols) && !small_path && !narrow;
    ColsPlan cols{};
    int grid_S = S;         // reduction splits as workgroups (S: as partial results)
    if (cols_path) {
        if (S > 1 && (!ws || ws_bytes < static_cast<size_t>(S) * M * N * sizeof(float)))
            CG_FAIL(CAPGNN_ENOMEM, "gemm: workspace of %zu bytes needed, %zu given", static_cast<size_t>(S) * M * N * sizeof(float), ws_bytes);
        cols = cols_plan(half_cols, M, N, K, S);
        grid_S = cols.S;
        S = cols.S * cols.parts;
        bn = 32 * cols.tb;
    }
    if (mid_path || (half_path && !trans_a && !small_path && tiles128 <= 1280)) bm = bn = 64;
    GemmArgs g;
    g.M = M; g.N = N; g.K = K;
    g.A = static_cast<const char *>(A); g.lda = lda;
    g.B = static_cast<const char *>(B); g.ldb = ldb;
    g.C = static_cast<char *>(C); g.ldc = ldc;
    g.part = nullptr;
    g.k_chunk = K > 0 ? K : 1;
    const size_t va = 4 * es;   // bytes of one 4-element vector
    g.a_vec = (reinterpret_cast<uintptr_t>(A) % va == 0) && ((lda * es) % va == 0);
    g.b_vec = (reinterpret_cast<uintptr_t>(B) % va == 0) && ((ldb * es) % va == 0);
    g.out_bf16 = (dtype == CAPGNN_BF16 && !out_f32);
    g.accumulate = accumulate; g.relu = relu; g.bias = bias;
    g.mask = static_cast<const char *>(relu_mask); g.ldm = ldm; g.mask_bf16 = (dtype == CAPGNN_BF16);
    g.rscale = row_scale;
    g.A2 = nullptr; g.lda2 = 0; g.K1 = 0; g.K1p = 0;
    if (S > 1) {
        const size_t need = static_cast<size_t>(S) * M * N * sizeof(float);
        if (!ws || ws_bytes < need) CG_FAIL(CAPGNN_ENOMEM, "gemm: workspace of %zu bytes needed, %zu given", need, ws_bytes);
        g.part = static_cast<float *>(ws);
        const int64_t steps = (K + bk - 1) / bk;
        g.k_chunk = (steps + S - 1) / S * bk;
    }
    if (small_path) g.k_chunk = small_chunk;
    if (cols_path) g.k_chunk = cols.chunk;
    if (narrow) {
        g.part = static_cast<float *>(ws);
        g.k_chunk = ((K + S - 1) / S + 15) / 16 * 16;      // (the last splits may be empty: zeros)
    }
    g.colpart = nullptr;
    if (colsum) {
        const size_t at = S > 1 || narrow ? align_up(static_cast<size_t>(S) * M * N * sizeof(float), 256) : 0;
        const size_t need = at + static_cast<size_t>(S) * N * sizeof(float);
        if (!ws || ws_bytes < need) CG_FAIL(CAPGNN_ENOMEM, "gemm: workspace of %zu bytes needed, %zu given", need, ws_bytes);
        g.colpart = reinterpret_cast<float *>(static_cast<char *>(ws) + at);
    }
    const int64_t gy = (M + bm - 1) / bm, gx = (N + bn - 1) / bn;
    if (!cols_path) grid_S = S;
    const int64_t n_wg = cols_path ? cols_grid(cols, M, N)
                         : grid_S > 1 ? NUM_XCD * ((grid_S + NUM_XCD - 1) / NUM_XCD) * gx * gy : NUM_XCD * ((gy + NUM_XCD - 1) / NUM_XCD) * gx;
    if (n_wg >= (int64_t(1) << 31) || gx >= (int64_t(1) << 24) || gy >= (int64_t(1) << 30))
        CG_FAIL(CAPGNN_EINVAL, "gemm: %lld x %lld tiles exceed the grid", (long long)gy, (long long)gx);
    g.gx = static_cast<int>(gx); g.gy = static_cast<int>(gy); g.S = grid_S;
    g.c_staged = half_path && g.out_bf16 && !g.part && !g.accumulate && !g.rscale && aligned16(C) && (ldc * 2) % 16 == 0 &&
                 (!relu_mask || (aligned16(relu_mask) && (ldm * 2) % 16 == 0));
    const bool stream_path = g.c_staged && !trans_a && bf16_stream_pays(M, N, K, relu_mask != nullptr) && ws &&
                             ws_bytes >= stream_b_bytes(N, K) && lda < (1 << 22) && ldc < (1 << 22) && ldm < (1 << 22);
    dim3 grid(static_cast<unsigned>(n_wg), 1, 1);
    bool akc = !trans_a, bkc = trans_b != 0;
    // nothing follows the product here: its parts, if any, are added up later
    const bool parts = S > 1 || colsum || narrow, alone = !parts || (later && reduce_later(later, g, S, nullptr, nullptr, 0, colsum));
    if (narrow) {
        SmallGemmArgs sm{};
        sm.g = g;
        launch_narrow(sm, grid, stream);
    } else if (small_path) {
        SmallGemmArgs sm{};
        sm.g = g;
        sm.M2 = M;
        if (!(alone && batch_small(batch, sm, dtype == CAPGNN_BF16, akc, bkc, tn, grid))) launch_small(sm, dtype == CAPGNN_BF16, akc, bkc, tn, grid, stream);
    } else if (mid_path) {
        SmallGemmArgs sm{};
        sm.g = g;
        sm.M2 = M;
        if (quarters) launch_quarters(sm, bkc, grid, stream);
        else if (bkc) hipLaunchKernelGGL(gemm_split_mid_kernel<true>, grid, dim3(256), 0, stream, sm);
        else hipLaunchKernelGGL(gemm_split_mid_kernel<false>, grid, dim3(256), 0, stream, sm);
    } else if (split_path) {
        if (trans_a) {
            SmallGemmArgs sm{};
            sm.g = g;
            launch_cols(sm, false, cols, grid, stream);
        } else {
            const int64_t n_pad = split_rows(N), ku_total = split_ld(K) / 8;
            hipLaunchKernelGGL(split_repack_kernel, dim3(static_cast<unsigned>((ku_total * n_pad * 8 + 255) / 256)), dim3(256), 0,
                               stream, static_cast<const float *>(B), ldb, bkc ? 1 : 0, K, N, static_cast<uint16_t *>(ws), n_pad,
                               ku_total);
            if (!launch_split_stream(g, static_cast<const uint16_t *>(ws), ku_total, n_pad, stream))
                launch_split_tiles(g, bn, grid, static_cast<const uint16_t *>(ws), ku_total, n_pad, stream);
        }
    } else if (stream_path) {
        const int64_t n_pad = split_rows(N), ku_total = 2 * stream_units(K);
        hipLaunchKernelGGL(unit_repack_kernel, dim3(static_cast<unsigned>((ku_total * n_pad * 8 + 255) / 256)), dim3(256), 0, stream,
                           static_cast<const uint16_t *>(B), ldb, bkc ? 1 : 0, K, N, static_cast<uint16_t *>(ws), n_pad, ku_total);
        launch_stream(g, static_cast<const uint16_t *>(ws), static_cast<uint32_t>(n_pad), stream);
    } else if (cols_path) {
        SmallGemmArgs sm{};
        sm.g = g;
        launch_cols(sm, true, cols, grid, stream);
    } else if (half_path) {
        if (repack_b) {
            const int64_t ldt = (K + 7) / 8 * 8;
            hipLaunchKernelGGL(repack_bf16_kernel, dim3(static_cast<unsigned>((N * ldt + 255) / 256)), dim3(256), 0, stream,
                               static_cast<const uint16_t *>(B), ldb, bkc ? 1 : 0, K, N, static_cast<uint16_t *>(ws), ldt);
            g.B = static_cast<const char *>(ws); g.ldb = ldt;
            bkc = true;
        }
        if (akc && bkc) launch_bf16_tiles<true, true>(g, bn, bm == 64, grid, stream);
        else if (akc) launch_bf16_tiles<true, false>(g, bn, bm == 64, grid, stream);
        else launch_bf16_tiles<false, true>(g, bn, bm == 64, grid, stream);
    } else {
        const bool bf = dtype == CAPGNN_BF16;
#define CG_GEMM_CASE(BF, AK, BKC_) if (bf == BF && akc == AK && bkc == BKC_) launch_tiles<BF, AK, BKC_>(g, bn, grid, stream);
        CG_GEMM_CASE(false, true, false) CG_GEMM_CASE(false, true, true)
        CG_GEMM_CASE(false, false, false) CG_GEMM_CASE(false, false, true)
        CG_GEMM_CASE(true, true, false) CG_GEMM_CASE(true, true, true)
        CG_GEMM_CASE(true, false, false) CG_GEMM_CASE(true, false, true)
#undef CG_GEMM_CASE
    }
    CG_HIP(hipGetLastError());
    if (!alone) {
        const int64_t blocks = (S > 1 || narrow ? (M * N + 31) / 32 : 0) + (colsum ? (N + 31) / 32 : 0);
        hipLaunchKernelGGL(gemm_reduce_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, g, S,
                           static_cast<const float *>(nullptr), static_cast<char *>(nullptr), int64_t(0), colsum);
        CG_HIP(hipGetLastError());
    }
    return CAPGNN_OK;
}

// Two products in one launch of gemm_small_kernel or gemm_split_mid_kernel: their sum C = op(A) op(B) + op(A2) op(B2) (dual), or
// C = op(A) op(B) and C2 = op(A2) op(B2) of one shape but for the rows (pair).  *done says whether the sizes are such a kernel's;
// nothing has run otherwise.
static int launch_two_small(const SmallGemmArgs &in, int trans_a, int trans_b, int dtype, int out_f32, void *ws, size_t ws_bytes,
                            hipStream_t stream, int f32_product, float *colsum, bool *done, FinishList *later = nullptr,
                            SmallBatch *batch = nullptr) {
    *done = false;
    SmallGemmArgs s = in;
    GemmArgs &g = s.g;
    const bool bf = dtype == CAPGNN_BF16, pair = s.C2 != nullptr;
    const int64_t Ksum = g.K + (s.dual ? s.K2 : 0);       // (the waves of a workgroup share it)
    // (a bf16 sum is two launches at every size: see launch_gemm_dual)
    const bool small = (bf ? !s.dual : f32_product != CAPGNN_F32_PRODUCT_SPLIT) && small_product(bf, trans_a, g.M, g.N, Ksum, s.dual || bf ? 2 : 1, trans_b);
    // two narrow reductions over vertices
    const size_t half_ws = ws_bytes / 2 / 256 * 256;
    const bool narrow = pair && g.M == s.M2 && ws && narrow_product(dtype, f32_product, trans_a, trans_b, g.M, g.N, g.K) &&
                        half_ws >= narrow_ws_bytes(g.M, g.N, g.K);
    // two reductions over vertices with the operands in registers, on the terms of launch_gemm
    auto rows16 = [](const void *p, int64_t ld) { return aligned16(p) && ld % 8 == 0; };
    const int most = choose_split(trans_a, g.M, g.N, g.K, 128, g.N <= 64 ? 64 : 128, HBK);
    const bool cols_pair = pair && trans_a && !trans_b && g.M == s.M2 && ws && !narrow && g.K > 0 && most > 1 && cols_reach(g.K, std::max(g.lda, s.lda2), g.ldb) &&
                           g.B == s.B2 && g.ldb == s.ldb2 && half_ws >= align_up(static_cast<size_t>(most) * g.M * g.N * sizeof(float), 256) + most * g.N * sizeof(float) &&
                           (bf ? rows16(g.A, g.lda) && rows16(s.A2, s.lda2) && rows16(g.B, g.ldb) && (!small || bf16_cols_pays(g.M, g.N, g.K))
                               : !small && split_form(f32_product, 1, g.M, g.N, g.K));
    if (cols_pair) {
        const ColsPlan cols = cols_plan(bf, g.M, g.N, g.K, most, 2);
        const int S = cols.S * cols.parts;
        g.k_chunk = cols.chunk;
        if (S > 1) {
            g.part = static_cast<float *>(ws);
            s.part2 = reinterpret_cast<float *>(static_cast<char *>(ws) + half_ws);
        }
        if (colsum) g.colpart = reinterpret_cast<float *>(static_cast<char *>(ws) + align_up(static_cast<size_t>(S) * g.M * g.N * sizeof(float), 256));
        g.out_bf16 = bf && !out_f32;
        g.gx = static_cast<int>((g.N + 32 * cols.tb - 1) / (32 * cols.tb)); g.gy = static_cast<int>((g.M + 127) / 128); g.S = cols.S;
        launch_cols(s, bf, cols, dim3(static_cast<unsigned>(cols_grid(cols, g.M, g.N)), 2, 1), stream);
        if ((S > 1 || colsum) && !(later && reduce_later(later, g, S, s.part2, s.C2, s.ldc2, colsum)))
            hipLaunchKernelGGL(gemm_reduce_kernel, dim3(static_cast<unsigned>((S > 1 ? (g.M * g.N + 31) / 32 : 0) + (colsum ? (g.N + 31) / 32 : 0)), 2), dim3(256), 0,
                               stream, g, S, static_cast<const float *>(s.part2), s.C2, s.ldc2, colsum);
        CG_HIP(hipGetLastError());
        *done = true;
        return CAPGNN_OK;
    }
    const int64_t tiles64 = ((g.M + 63) / 64) * ((g.N + 63) / 64);
    // the three-piece form on the terms of launch_gemm and launch_gemm_dual
    const bool split = !bf && !trans_a && ws && ws_bytes >= split_b_bytes(g.N, s.dual ? split_ld(g.K) + s.K2 : g.K) &&
                       (s.dual ? split_sum(f32_product, trans_b, g.M, g.N, g.K, s.K2)
                               : split_form(f32_product, 0, g.M, g.N, g.K) && split_form(f32_product, 0, s.M2, g.N, g.K));
    const bool mid = !small && split && tiles64 * (pair ? 2 : 1) <= 768 &&
                     std::max(std::max(g.lda, s.lda2), std::max(g.ldb, s.ldb2)) < (1 << 22);
    if ((!small && !mid && !narrow) || g.K <= 0 || (s.dual && s.K2 <= 0)) return CAPGNN_OK;
    int tn = 2, S = 1;
    g.k_chunk = Ksum;
    if (narrow) {
        S = narrow_splits(g.M, g.K);
        g.k_chunk = ((g.K + S - 1) / S + 15) / 16 * 16;
        g.part = static_cast<float *>(ws);
        s.part2 = reinterpret_cast<float *>(static_cast<char *>(ws) + half_ws);
        if (colsum) g.colpart = g.part + align_up(static_cast<size_t>(S) * g.M * g.N * sizeof(float), 256) / sizeof(float);
    } else if (small) small_geometry(bf, trans_a, g.M, g.N, g.K, &tn, &S, &g.k_chunk);
    if (s.dual && S > 1) return CAPGNN_OK;           // a sum is formed by the waves of one workgroup
    if (narrow) {
    } else if (S > 1) {
        const size_t one = align_up(static_cast<size_t>(S) * g.M * g.N * sizeof(float), 256);
        if (g.M != s.M2 || !ws || ws_bytes < 2 * one + static_cast<size_t>(S) * g.N * sizeof(float)) return CAPGNN_OK;
        g.part = static_cast<float *>(ws);
        s.part2 = reinterpret_cast<float *>(static_cast<char *>(ws) + one);
        if (colsum) g.colpart = reinterpret_cast<float *>(static_cast<char *>(ws) + 2 * one);
    } else if (colsum) {
        if (!ws || ws_bytes < g.N * sizeof(float)) return CAPGNN_OK;
        g.colpart = static_cast<float *>(ws);
    }
    const int es = elem_bytes(dtype);
    auto vec_rows = [&](const void *p, int64_t ld) { return reinterpret_cast<uintptr_t>(p) % (4 * es) == 0 && (ld * es) % (4 * es) == 0; };
    g.a_vec = vec_rows(g.A, g.lda) && vec_rows(s.A2, s.lda2);
    g.b_vec = vec_rows(g.B, g.ldb) && vec_rows(s.B2, s.ldb2);
    g.out_bf16 = bf && !out_f32;
    const int bm = narrow ? 128 : small ? 32 : 64, bn = narrow || !small ? 64 : 32 * tn;
    const int64_t gy = (std::max(g.M, s.M2) + bm - 1) / bm, gx = (g.N + bn - 1) / bn;
    g.gx = static_cast<int>(gx); g.gy = static_cast<int>(gy); g.S = S;
    const int64_t n_wg = S > 1 ? NUM_XCD * ((S + NUM_XCD - 1) / NUM_XCD) * gx * gy : NUM_XCD * ((gy + NUM_XCD - 1) / NUM_XCD) * gx;
    const dim3 grid(static_cast<unsigned>(n_wg), pair ? 2 : 1, 1);
    const bool alone = !(S > 1 || colsum || narrow) || (later && reduce_later(later, g, S, pair ? s.part2 : nullptr, s.C2, s.ldc2, colsum));
    if (narrow) launch_narrow(s, grid, stream);
    else if (small && alone && batch_small(batch, s, bf, !trans_a, trans_b != 0, tn, grid)) {}
    else if (small) launch_small(s, bf, !trans_a, trans_b != 0, tn, grid, stream);
    else if (quarters_pay(pair ? g.M + s.M2 : g.M, g.N, Ksum, trans_b)) launch_quarters(s, trans_b != 0, grid, stream);
    else if (trans_b) hipLaunchKernelGGL(gemm_split_mid_kernel<true>, grid, dim3(256), 0, stream, s);
    else hipLaunchKernelGGL(gemm_split_mid_kernel<false>, grid, dim3(256), 0, stream, s);
    if (!alone)
        hipLaunchKernelGGL(gemm_reduce_kernel,
                           dim3(static_cast<unsigned>((S > 1 || narrow ? (g.M * g.N + 31) / 32 : 0) + (colsum ? (g.N + 31) / 32 : 0)), pair ? 2 : 1),
                           dim3(256), 0, stream, g, S, static_cast<const float *>(s.part2), s.C2, s.ldc2, colsum);
    CG_HIP(hipGetLastError());
    *done = true;
    return CAPGNN_OK;
}

// C = op(A) op(B), C2 = op(A2) op(B2): the neighbour and self products of a GraphSAGE layer's backward pass (weight gradients: one
// second operand; input gradients: one first operand) or of its forward pass in the transform-first order (M rows and M2 <= M).
int launch_gemm_pair(int trans_a, int trans_b, int64_t M, int64_t M2, int64_t N, int64_t K, const void *A, int64_t lda, const void *A2,
                     int64_t lda2, const void *B, int64_t ldb, const void *B2, int64_t ldb2, void *C, int64_t ldc, void *C2,
                     int64_t ldc2, int dtype, int out_f32, const float *row_scale, void *ws, size_t ws_bytes, hipStream_t stream,
                     int f32_product, float *colsum, FinishList *later, SmallBatch *batch) {
    if (M2 > M) CG_FAIL(CAPGNN_EINVAL, "gemm_pair: the second product has more rows");
    if (f32_product != CAPGNN_F32_PRODUCT_AUTO && f32_product != CAPGNN_F32_PRODUCT_NATIVE && f32_product != CAPGNN_F32_PRODUCT_SPLIT)
        CG_FAIL(CAPGNN_EINVAL, "gemm: unknown form of the fp32 product %d", f32_product);
    SmallGemmArgs s{};
    s.g.M = M; s.g.N = N; s.g.K = K;
    s.g.A = static_cast<const char *>(A); s.g.lda = lda; s.g.B = static_cast<const char *>(B); s.g.ldb = ldb;
    s.g.C = static_cast<char *>(C); s.g.ldc = ldc; s.g.rscale = row_scale;
    s.A2 = static_cast<const char *>(A2); s.lda2 = lda2; s.B2 = static_cast<const char *>(B2); s.ldb2 = ldb2;
    s.C2 = static_cast<char *>(C2); s.ldc2 = ldc2; s.M2 = M2;
    bool done = false;
    // results that share memory are written one after the other, as the two launches do
    const int64_t es_c = (dtype == CAPGNN_BF16 && !out_f32) ? 2 : 4;
    const uintptr_t c1 = reinterpret_cast<uintptr_t>(C), c2 = reinterpret_cast<uintptr_t>(C2);
    const bool apart = c1 + ((M - 1) * ldc + N) * es_c <= c2 || c2 + ((M2 - 1) * ldc2 + N) * es_c <= c1;
    // (the sum over splits scales both results alike, and row_scale is the first one's)
    if (apart && !(trans_a && row_scale) && M2 > 0 && N > 0 && A && A2 && B && B2 && C && C2 && ldc >= N && ldc2 >= N && lda >= (trans_a ? M : K) &&
        lda2 >= (trans_a ? M : K) && ldb >= (trans_b ? K : N) && ldb2 >= (trans_b ? K : N))
        CG_TRY(launch_two_small(s, trans_a, trans_b, dtype, out_f32, ws, ws_bytes, stream, f32_product, colsum, &done, later, batch));
    if (done) return CAPGNN_OK;
    // (parts that are added up later keep half of the workspace each)
    const size_t half = later ? ws_bytes / 2 / 256 * 256 : 0;
    CG_TRY(launch_gemm(trans_a, trans_b, M, N, K, A, lda, B, ldb, C, ldc, dtype, out_f32, 0, nullptr, 0, nullptr, 0, ws,
                       later ? half : ws_bytes, stream, row_scale, f32_product, colsum, later, batch));
    return launch_gemm(trans_a, trans_b, M2, N, K, A2, lda2, B2, ldb2, C2, ldc2, dtype, out_f32, 0, nullptr, 0, nullptr, 0,
                       ws ? static_cast<char *>(ws) + half : nullptr, ws_bytes - half, stream, nullptr, f32_product, nullptr, later, batch);
}

size_t gemm_pair_ws_bytes(int trans_a, int64_t M, int64_t N, int64_t K) { return (trans_a ? 2 : 1) * gemm_ws_bytes(trans_a, M, N, K); }

// C = A op(W) + A2 op(W2) (+ bias, ReLU): the two products of a GraphSAGE layer (neighbour term and self term), or of its input
// gradient, into one result.  fp32 operands of small and middling sizes, and in the three-piece form, run as ONE launch, whose
// reduction walks both first operands, so C is written once and never read back; every other case is the two launches it
// replaces (A2 W2 first, then A W accumulated on top with the epilogue).  bf16 operands are always two: A2 W2 is rounded as it is
// stored, at every number of rows alike.  One launch for few rows, rounding once, moved the gradients of layers of 1000 to 4000 vertices by 2
// to 5 % of their norm (pre-activations near zero change sides).  A [M x K1], A2 [M x K2] row-major; W [K1 x N], W2 [K2 x N], or
// their transposes when trans_b.
int launch_gemm_dual(int trans_b, int64_t M, int64_t N, int64_t K1, const void *A, int64_t lda, const void *W, int64_t ldw, int64_t K2,
                     const void *A2, int64_t lda2, const void *W2, int64_t ldw2, void *C, int64_t ldc, int dtype, int out_f32,
                     const float *bias, int relu, void *ws, size_t ws_bytes, hipStream_t stream, int f32_product, const void *relu_mask,
                     int64_t ldm, SmallBatch *batch) {
    if (f32_product != CAPGNN_F32_PRODUCT_AUTO && f32_product != CAPGNN_F32_PRODUCT_NATIVE && f32_product != CAPGNN_F32_PRODUCT_SPLIT)
        CG_FAIL(CAPGNN_EINVAL, "gemm: unknown form of the fp32 product %d", f32_product);
    const bool sane = M > 0 && N > 0 && K1 > 0 && K2 > 0 && A && A2 && W && W2 && C && lda >= K1 && lda2 >= K2 &&
                      ldw >= (trans_b ? K1 : N) && ldw2 >= (trans_b ? K2 : N) && ldc >= N && N <= (1 << 22) &&
                      M < (int64_t(1) << 31) * 64;
    GemmArgs g{};
    g.M = M; g.N = N;
    g.A = static_cast<const char *>(A); g.lda = lda;
    g.B = static_cast<const char *>(W); g.ldb = ldw;
    g.C = static_cast<char *>(C); g.ldc = ldc;
    g.relu = relu; g.bias = bias;
    g.mask = static_cast<const char *>(relu_mask); g.ldm = ldm; g.mask_bf16 = dtype == CAPGNN_BF16;
    if (sane) {
        SmallGemmArgs s{};
        s.g = g;
        s.g.K = K1; s.K2 = K2; s.dual = 1; s.M2 = M;
        s.A2 = static_cast<const char *>(A2); s.lda2 = lda2; s.B2 = static_cast<const char *>(W2); s.ldb2 = ldw2;
        bool done = false;
        CG_TRY(launch_two_small(s, 0, trans_b, dtype, out_f32, ws, ws_bytes, stream, f32_product, nullptr, &done, nullptr, batch));
        if (done) return CAPGNN_OK;
    }
    const int64_t K1p = split_ld(K1 > 0 ? K1 : 0), K = K1p + K2;
    const bool one_launch = sane && dtype == CAPGNN_F32 && lda < (1 << 22) && lda2 < (1 << 22) &&
                            split_sum(f32_product, trans_b, M, N, K1, K2) && ws && ws_bytes >= split_b_bytes(N, K);
    if (!one_launch) {
        CG_TRY(launch_gemm(0, trans_b, M, N, K2, A2, lda2, W2, ldw2, C, ldc, dtype, out_f32, 0, nullptr, 0, nullptr, 0, ws, ws_bytes,
                           stream, nullptr, f32_product));
        return launch_gemm(0, trans_b, M, N, K1, A, lda, W, ldw, C, ldc, dtype, out_f32, 1, bias, relu, relu_mask, ldm, ws, ws_bytes,
                           stream, nullptr, f32_product);
    }
    int bm, bn;
    tile_for(N, &bm, &bn);
    g.K = K;
    g.k_chunk = K;
    g.a_vec = (reinterpret_cast<uintptr_t>(A) % 16 == 0) && ((lda * 4) % 16 == 0) && (reinterpret_cast<uintptr_t>(A2) % 16 == 0) &&
              ((lda2 * 4) % 16 == 0);
    g.A2 = static_cast<const char *>(A2); g.lda2 = lda2; g.K1 = K1; g.K1p = K1p;
    const int64_t gy = (M + bm - 1) / bm, gx = (N + bn - 1) / bn;
    const int64_t n_wg = NUM_XCD * ((gy + NUM_XCD - 1) / NUM_XCD) * gx;
    if (n_wg >= (int64_t(1) << 31) || gx >= (int64_t(1) << 24) || gy >= (int64_t(1) << 30))
        CG_FAIL(CAPGNN_EINVAL, "gemm: %lld x %lld tiles exceed the grid", (long long)gy, (long long)gx);
    g.gx = static_cast<int>(gx); g.gy = static_cast<int>(gy); g.S = 1;
    const int64_t n_pad = split_rows(N), ku_total = split_ld(K) / 8;
    hipLaunchKernelGGL(split_repack_kernel, dim3(static_cast<unsigned>((ku_total * n_pad * 8 + 255) / 256)), dim3(256), 0, stream,
                       static_cast<const float *>(W), ldw, trans_b ? 1 : 0, K1, N, static_cast<uint16_t *>(ws), n_pad, ku_total,
                       static_cast<const float *>(W2), ldw2, K1p, K2);
    dim3 grid(static_cast<unsigned>(n_wg), 1, 1);
    if (launch_split_stream(g, static_cast<const uint16_t *>(ws), ku_total, n_pad, stream)) {
    } else if (bn == 64)
        hipLaunchKernelGGL((gemm_split_kernel<128, 64, 4, true>), grid, dim3(256), 0, stream, g, static_cast<const uint16_t *>(ws),
                           ku_total, n_pad);
    else
        hipLaunchKernelGGL((gemm_split_kernel<128, 128, 8, true>), grid, dim3(512), 0, stream, g, static_cast<const uint16_t *>(ws),
                           ku_total, n_pad);
    CG_HIP(hipGetLastError());
    return CAPGNN_OK;
}

// Register-resident matrix-instruction loop: what the matrix cores deliver on this chip when nothing else is in
// the way (four independent 32x32 accumulator tiles per wave, operands never reloaded).  The utilisation figures
// of the product kernels can be read against it as well as against the data-sheet peak.
template <bool BF16>
__global__ __launch_bounds__(256) void mfma_peak_kernel(int iters, float *out) {
    floatx16 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    const float a = 1.f + 1e-3f * threadIdx.x, b = 1.f - 1e-3f * threadIdx.x;
    bf16x8 ha, hb;
#pragma unroll
    for (int j = 0; j < 8; ++j) { ha[j] = static_cast<__bf16>(a); hb[j] = static_cast<__bf16>(b); }
    for (int i = 0; i < iters; ++i) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if constexpr (BF16) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ha, hb, acc[t], 0, 0, 0);
            else acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[t], 0, 0, 0);
        }
    }
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += acc[t][r];
    out[static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x] = s;     // keeps the loop alive
}

}  // namespace capgnn

using namespace capgnn;

extern "C" int capgnn_mfma_peak(int dtype, int workgroups, int iters, float *out, double *flop, void *stream) {
    if ((dtype != CAPGNN_F32 && dtype != CAPGNN_BF16) || workgroups <= 0 || iters <= 0 || !out || !flop)
        CG_FAIL(CAPGNN_EINVAL, "mfma_peak: bad argument");
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (dtype == CAPGNN_BF16) hipLaunchKernelGGL(mfma_peak_kernel<true>, dim3(workgroups), dim3(256), 0, st, iters, out);
    else hipLaunchKernelGGL(mfma_peak_kernel<false>, dim3(workgroups), dim3(256), 0, st, iters, out);
    CG_HIP(hipGetLastError());
    const double per_instr = dtype == CAPGNN_BF16 ? 2.0 * 32 * 32 * 16 : 2.0 * 32 * 32 * 2;
    *flop = per_instr * 4.0 * iters * 4.0 * workgroups;     // 4 tiles per wave, 4 waves per workgroup
    return CAPGNN_OK;
}

extern "C" size_t capgnn_gemm_workspace_bytes(int trans_a, int64_t M, int64_t N, int64_t K) {
    return gemm_ws_bytes(trans_a, M, N, K);
}

extern "C" int capgnn_gemm(int trans_a, int trans_b, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
                           const void *B, int64_t ldb, void *C, int64_t ldc, int dtype, int out_f32, int accumulate,
                           const float *bias, int relu, const void *relu_mask, int64_t ldm, int f32_product, void *ws,
                           size_t ws_bytes, void *stream) {
    return launch_gemm(trans_a, trans_b, M, N, K, A, lda, B, ldb, C, ldc, dtype, out_f32, accumulate, bias, relu,
                       relu_mask, ldm, ws, ws_bytes, static_cast<hipStream_t>(stream), nullptr, f32_product);
}
