// Small VALU kernels around the layer: sigma' masking + bias gradient, softmax cross-entropy, SGD step.
#include "common.h"

#include <mutex>

#include <algorithm>

namespace capgnn {

__device__ __forceinline__ float ld_elem(const char *p, int64_t i, int bf16) {
    return bf16 ? __uint_as_float(static_cast<uint32_t>(reinterpret_cast<const uint16_t *>(p)[i]) << 16)
                : reinterpret_cast<const float *>(p)[i];
}

__device__ __forceinline__ void st_elem(char *p, int64_t i, float v, int bf16) {
    if (bf16) {
        uint32_t u = __float_as_uint(v);
        if ((u & 0x7fffffffu) > 0x7f800000u) u = (u >> 16) | 0x40u;
        else u = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
        reinterpret_cast<uint16_t *>(p)[i] = static_cast<uint16_t>(u);
    } else {
        reinterpret_cast<float *>(p)[i] = v;
    }
}

// ------------------------------------------------------------------ dZ = dH * 1[H>0], dbias partials
constexpr int RB_ROWS = 128;          // rows per chunk
constexpr int RB_MAX_BLOCKS = 1024;   // workgroups (= partial rows); each walks chunks b, b+grid, ...

// blockDim = (TX, 256/TX): threadIdx.x walks the feature columns, threadIdx.y the rows of a chunk.
// dst = src * 1[H > 0] (all of src when !relu), written in place (only the zeroed elements are stored) or,
// when dst differs from src, as a converting copy.  partial[b][f] = this workgroup's column sums of dst,
// formed from the unrounded values.
__global__ __launch_bounds__(256) void relu_mask_dbias_kernel(int64_t n, int F, const char *src, int64_t lds,
                                                              int src_bf16, char *dst, int64_t ldd, int dst_bf16,
                                                              const char *H, int64_t ldh, int h_bf16, int relu,
                                                              float *partial, const float *rscale) {
    __shared__ float red[256];
    const int tx = threadIdx.x, ty = threadIdx.y, TX = blockDim.x, TY = blockDim.y;
    const bool in_place = src == dst;
    for (int f0 = 0; f0 < F; f0 += TX) {
        const int f = f0 + tx;
        float s = 0.f;
        if (f < F) {
            for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * RB_ROWS; r0 < n; r0 += static_cast<int64_t>(gridDim.x) * RB_ROWS) {
                const int64_t r1 = r0 + RB_ROWS < n ? r0 + RB_ROWS : n;
                for (int64_t r = r0 + ty; r < r1; r += TY) {
                    float g = ld_elem(src, r * lds + f, src_bf16);
                    bool zeroed = false;
                    if (relu) {
                        const float h = ld_elem(H, r * ldh + f, h_bf16);
                        if (!(h > 0.f)) { g = 0.f; zeroed = true; }
                    }
                    s += g;
                    if (rscale) g *= rscale[r];         // the stored copy carries the row's scale, the column sums do not
                    if (!in_place || zeroed || rscale) st_elem(dst, r * ldd + f, g, dst_bf16);
                }
            }
        }
        if (partial) {
            red[ty * TX + tx] = s;
            __syncthreads();
            if (ty == 0 && f < F) {
                float t = 0.f;
                for (int y = 0; y < TY; ++y) t += red[y * TX + tx];
                partial[static_cast<int64_t>(blockIdx.x) * F + f] = t;
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ float4 ld4(const char *p, int64_t i, int bf16) {
    if (bf16) {
        const uint2 v = *reinterpret_cast<const uint2 *>(reinterpret_cast<const uint16_t *>(p) + i);
        return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                           __uint_as_float(v.y & 0xffff0000u));
    }
    return *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(p) + i);
}

__device__ __forceinline__ uint32_t bf16_rne_bits(float v) {
    uint32_t u = __float_as_uint(v);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// The same operation with four consecutive features per thread (8- or 16-byte accesses); needs rows that start on
// 16-byte boundaries.  blockDim = (TX, 256/TX), TX = ceil(F/4) rounded up to a power of two (F <= 1024).
__global__ __launch_bounds__(256) void relu_mask_dbias_vec4_kernel(int64_t n, int F, const char *src, int64_t lds,
                                                                   int src_bf16, char *dst, int64_t ldd, int dst_bf16,
                                                                   const char *H, int64_t ldh, int h_bf16, int relu,
                                                                   float *partial, const float *rscale) {
    __shared__ float red[256][4];
    const int tx = threadIdx.x, ty = threadIdx.y, TX = blockDim.x, TY = blockDim.y;
    const bool in_place = src == dst;
    const int f = 4 * tx;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (f < F) {
        const int nv = F - f < 4 ? F - f : 4;    // valid features of this thread's vector (the rest is row padding)
        for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * RB_ROWS; r0 < n; r0 += static_cast<int64_t>(gridDim.x) * RB_ROWS) {
            const int64_t r1 = r0 + RB_ROWS < n ? r0 + RB_ROWS : n;
            // four rows per trip: their loads are issued together, so a thread keeps eight vectors in flight
            for (int64_t rb = r0 + ty; rb < r1; rb += 4 * TY) {
                float4 gv[4], hv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t r = rb + static_cast<int64_t>(u) * TY;
                    if (r < r1) {
                        gv[u] = ld4(src, r * lds + f, src_bf16);
                        if (relu) hv[u] = ld4(H, r * ldh + f, h_bf16);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t r = rb + static_cast<int64_t>(u) * TY;
                    if (r >= r1) continue;
                    float g[4] = {gv[u].x, gv[u].y, gv[u].z, gv[u].w};
                    bool zeroed = false;
                    if (relu) {
                        const float h[4] = {hv[u].x, hv[u].y, hv[u].z, hv[u].w};
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (!(h[j] > 0.f) && g[j] != 0.f) { g[j] = 0.f; zeroed = true; }
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j) s[j] += g[j];
                    if (rscale) {                       // the stored copy carries the row's scale, the column sums do not
                        const float rs = rscale[r];
#pragma unroll
                        for (int j = 0; j < 4; ++j) g[j] *= rs;
                    }
                    if (!in_place || zeroed || rscale) {
                        if (nv == 4) {
                            if (dst_bf16) {
                                uint2 o;
                                o.x = bf16_rne_bits(g[0]) | (bf16_rne_bits(g[1]) << 16);
                                o.y = bf16_rne_bits(g[2]) | (bf16_rne_bits(g[3]) << 16);
                                *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(dst) + r * ldd + f) = o;
                            } else {
                                *reinterpret_cast<float4 *>(reinterpret_cast<float *>(dst) + r * ldd + f) = make_float4(g[0], g[1], g[2], g[3]);
                            }
                        } else {
                            for (int j = 0; j < nv; ++j) st_elem(dst, r * ldd + f + j, g[j], dst_bf16);
                        }
                    }
                }
            }
        }
    }
    if (!partial) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) red[ty * TX + tx][j] = s[j];
    __syncthreads();
    if (ty == 0 && f < F) {
        for (int j = 0; j < 4 && f + j < F; ++j) {
            float t = 0.f;
            for (int y = 0; y < TY; ++y) t += red[y * TX + tx][j];
            partial[static_cast<int64_t>(blockIdx.x) * F + f + j] = t;
        }
    }
}

// The same for bf16 data on all three sides with eight consecutive features per thread (16-byte accesses): the wide
// bf16 layers are bound by this kernel's memory traffic, and 8-byte accesses leave half of the load path idle.
// blockDim = (TX, 256/TX), TX = ceil(F/8) rounded up to a power of two (F <= 2048); rows start on 16-byte boundaries.
__global__ __launch_bounds__(256) void relu_mask_dbias_bf16x8_kernel(int64_t n, int F, const char *src, int64_t lds, char *dst,
                                                                     int64_t ldd, const char *H, int64_t ldh, int relu,
                                                                     float *partial, const float *rscale) {
    __shared__ float red[256][8];
    const int tx = threadIdx.x, ty = threadIdx.y, TX = blockDim.x, TY = blockDim.y;
    const bool in_place = src == dst;
    const int f = 8 * tx;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (f < F) {
        const int nv = F - f < 8 ? F - f : 8;    // valid features of this thread's vector (the rest is row padding)
        for (int64_t r0 = static_cast<int64_t>(blockIdx.x) * RB_ROWS; r0 < n; r0 += static_cast<int64_t>(gridDim.x) * RB_ROWS) {
            const int64_t r1 = r0 + RB_ROWS < n ? r0 + RB_ROWS : n;
            for (int64_t rb = r0 + ty; rb < r1; rb += 4 * TY) {
                uint4 gv[4], hv[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t r = rb + static_cast<int64_t>(u) * TY;
                    if (r < r1) {
                        gv[u] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(src) + r * lds + f);
                        if (relu) hv[u] = *reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(H) + r * ldh + f);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t r = rb + static_cast<int64_t>(u) * TY;
                    if (r >= r1) continue;
                    const uint32_t gw[4] = {gv[u].x, gv[u].y, gv[u].z, gv[u].w};
                    float g[8];
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        g[2 * d] = __uint_as_float(gw[d] << 16);
                        g[2 * d + 1] = __uint_as_float(gw[d] & 0xffff0000u);
                    }
                    bool zeroed = false;
                    if (relu) {
                        const uint32_t hw[4] = {hv[u].x, hv[u].y, hv[u].z, hv[u].w};
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const float h0 = __uint_as_float(hw[d] << 16), h1 = __uint_as_float(hw[d] & 0xffff0000u);
                            if (!(h0 > 0.f) && g[2 * d] != 0.f) { g[2 * d] = 0.f; zeroed = true; }
                            if (!(h1 > 0.f) && g[2 * d + 1] != 0.f) { g[2 * d + 1] = 0.f; zeroed = true; }
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) s[j] += g[j];
                    if (rscale) {                       // the stored copy carries the row's scale, the column sums do not
                        const float rs = rscale[r];
#pragma unroll
                        for (int j = 0; j < 8; ++j) g[j] *= rs;
                    }
                    if (!in_place || zeroed || rscale) {
                        if (nv == 8) {
                            uint4 o;
                            o.x = bf16_rne_bits(g[0]) | (bf16_rne_bits(g[1]) << 16);
                            o.y = bf16_rne_bits(g[2]) | (bf16_rne_bits(g[3]) << 16);
                            o.z = bf16_rne_bits(g[4]) | (bf16_rne_bits(g[5]) << 16);
                            o.w = bf16_rne_bits(g[6]) | (bf16_rne_bits(g[7]) << 16);
                            *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(dst) + r * ldd + f) = o;
                        } else {
                            for (int j = 0; j < nv; ++j) st_elem(dst, r * ldd + f + j, g[j], 1);
                        }
                    }
                }
            }
        }
    }
    if (!partial) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) red[ty * TX + tx][j] = s[j];
    __syncthreads();
    if (ty == 0 && f < F) {
        for (int j = 0; j < 8 && f + j < F; ++j) {
            float t = 0.f;
            for (int y = 0; y < TY; ++y) t += red[y * TX + tx][j];
            partial[static_cast<int64_t>(blockIdx.x) * F + f + j] = t;
        }
    }
}

// dbias[f] = sum_b partial[b][f] for 32 features f from 32 * chunk on: 32 strided groups of 32 threads, doubles, fixed order.
// red: 1024 doubles of LDS.
constexpr int DBF_GROUPS = 32;
__device__ __forceinline__ void column_sums(int chunk, int64_t nblocks, int F, const float *partial, float *dbias, double *red) {
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int f = chunk * 32 + tx;
    double s = 0.0;
    if (f < F) {
        int64_t b = ty;
        for (; b + 3 * DBF_GROUPS < nblocks; b += 4 * DBF_GROUPS) {      // four loads in flight
            const float v0 = partial[b * F + f], v1 = partial[(b + DBF_GROUPS) * F + f];
            const float v2 = partial[(b + 2 * DBF_GROUPS) * F + f], v3 = partial[(b + 3 * DBF_GROUPS) * F + f];
            s += static_cast<double>(v0); s += static_cast<double>(v1);
            s += static_cast<double>(v2); s += static_cast<double>(v3);
        }
        for (; b < nblocks; b += DBF_GROUPS) s += static_cast<double>(partial[b * F + f]);
    }
    red[ty * 32 + tx] = s;
    __syncthreads();
    if (ty == 0 && f < F) {
        double t = 0.0;
        for (int y = 0; y < DBF_GROUPS; ++y) t += red[y * 32 + tx];
        dbias[f] = static_cast<float>(t);
    }
}

__global__ __launch_bounds__(1024) void dbias_final_kernel(int64_t nblocks, int F, const float *partial, float *dbias) {
    __shared__ double red[1024];
    column_sums(blockIdx.x, nblocks, F, partial, dbias, red);
}

static int64_t rb_blocks(int64_t n) {
    return std::max<int64_t>(1, std::min<int64_t>((n + RB_ROWS - 1) / RB_ROWS, RB_MAX_BLOCKS));
}

size_t relu_bias_ws_bytes(int64_t n, int F) {
    return align_up(static_cast<size_t>(rb_blocks(n)) * F * sizeof(float), 256);
}

int launch_relu_mask_dbias(int64_t n, int F, const void *src, int64_t lds, int src_dtype, void *dH, int64_t lddh,
                           const void *H, int64_t ldh, int dtype, int h_dtype, int relu, float *dbias, void *ws,
                           size_t ws_bytes, hipStream_t stream, const float *row_scale) {
    if (F <= 0) return CAPGNN_OK;
    if (n <= 0) {   // no rows: the bias gradient is zero (summing zero partial blocks)
        if (dbias) {
            hipLaunchKernelGGL(dbias_final_kernel, dim3((F + 31) / 32), dim3(32 * DBF_GROUPS), 0, stream, int64_t(0), F,
                               static_cast<const float *>(nullptr), dbias);
            CG_HIP(hipGetLastError());
        }
        return CAPGNN_OK;
    }
    if (!src) { src = dH; lds = lddh; src_dtype = dtype; }
    const bool converting = src != dH;
    if (!relu && !dbias && !converting && !row_scale) return CAPGNN_OK;
    if (!dH || (relu && !H)) CG_FAIL(CAPGNN_EINVAL, "relu_mask_dbias: NULL operand");
    if (lddh < F || lds < F || (relu && ldh < F)) CG_FAIL(CAPGNN_EINVAL, "relu_mask_dbias: leading dimension smaller than F");
    const int64_t nb = rb_blocks(n);
    if (dbias && (!ws || ws_bytes < static_cast<size_t>(nb) * F * sizeof(float)))
        CG_FAIL(CAPGNN_ENOMEM, "relu_mask_dbias: workspace too small");
    const int ses = elem_bytes(src_dtype), des = elem_bytes(dtype), hes = elem_bytes(h_dtype);
    const bool vec = F <= 1024 && aligned16(src) && aligned16(dH) && (lds * ses) % 16 == 0 && (lddh * des) % 16 == 0 &&
                     (!relu || (aligned16(H) && (ldh * hes) % 16 == 0));
    const bool all_bf16 = src_dtype == CAPGNN_BF16 && dtype == CAPGNN_BF16 && (!relu || h_dtype == CAPGNN_BF16);
    if (vec && all_bf16 && F >= 64 && F <= 2048) {
        int TX = 1;
        while (TX < (F + 7) / 8) TX <<= 1;
        dim3 block(TX, 256 / TX);
        hipLaunchKernelGGL(relu_mask_dbias_bf16x8_kernel, dim3(static_cast<unsigned>(nb)), block, 0, stream, n, F,
                           static_cast<const char *>(src), lds, static_cast<char *>(dH), lddh, static_cast<const char *>(H), ldh,
                           relu, dbias ? static_cast<float *>(ws) : nullptr, row_scale);
        CG_HIP(hipGetLastError());
        if (dbias) {
            hipLaunchKernelGGL(dbias_final_kernel, dim3((F + 31) / 32), dim3(32 * DBF_GROUPS), 0, stream, nb, F,
                               static_cast<const float *>(ws), dbias);
            CG_HIP(hipGetLastError());
        }
        return CAPGNN_OK;
    }
    if (vec) {
        int TX = 1;
        while (TX < (F + 3) / 4) TX <<= 1;
        dim3 block(TX, 256 / TX);
        hipLaunchKernelGGL(relu_mask_dbias_vec4_kernel, dim3(static_cast<unsigned>(nb)), block, 0, stream, n, F,
                           static_cast<const char *>(src), lds, src_dtype == CAPGNN_BF16 ? 1 : 0, static_cast<char *>(dH), lddh,
                           dtype == CAPGNN_BF16 ? 1 : 0, static_cast<const char *>(H), ldh, h_dtype == CAPGNN_BF16 ? 1 : 0,
                           relu, dbias ? static_cast<float *>(ws) : nullptr, row_scale);
        CG_HIP(hipGetLastError());
        if (dbias) {
            hipLaunchKernelGGL(dbias_final_kernel, dim3((F + 31) / 32), dim3(32 * DBF_GROUPS), 0, stream, nb, F,
                               static_cast<const float *>(ws), dbias);
            CG_HIP(hipGetLastError());
        }
        return CAPGNN_OK;
    }
    int TX = 1;
    while (TX < F && TX < 256) TX <<= 1;
    dim3 block(TX, 256 / TX);
    hipLaunchKernelGGL(relu_mask_dbias_kernel, dim3(static_cast<unsigned>(nb)), block, 0, stream, n, F,
                       static_cast<const char *>(src), lds, src_dtype == CAPGNN_BF16 ? 1 : 0, static_cast<char *>(dH), lddh,
                       dtype == CAPGNN_BF16 ? 1 : 0, static_cast<const char *>(H), ldh, h_dtype == CAPGNN_BF16 ? 1 : 0,
                       relu, dbias ? static_cast<float *>(ws) : nullptr, row_scale);
    CG_HIP(hipGetLastError());
    if (dbias) {
        hipLaunchKernelGGL(dbias_final_kernel, dim3((F + 31) / 32), dim3(32 * DBF_GROUPS), 0, stream, nb, F,
                           static_cast<const float *>(ws), dbias);
        CG_HIP(hipGetLastError());
    }
    return CAPGNN_OK;
}

// ------------------------------------------------------------------ SGD
// W -= lr * dW for all of a model's tensors in one launch: workgroups [first[t], first[t+1]) walk tensor t.
__global__ __launch_bounds__(256) void sgd_kernel(SgdList s, float lr) {
    int t = 0;
    while (t + 1 < s.count && blockIdx.x >= s.first[t + 1]) ++t;
    const int64_t blocks = (t + 1 < s.count ? s.first[t + 1] : gridDim.x) - s.first[t], b = blockIdx.x - s.first[t];
    float *W = s.W[t];
    const float *dW = s.dW[t];
    for (int64_t i = b * 256 + threadIdx.x; i < s.n[t]; i += blocks * 256) W[i] = W[i] - lr * dW[i];
}

static bool overlap(const float *a, int64_t na, const float *b, int64_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + nb * sizeof(float) && y < x + na * sizeof(float);
}

// The tensors of one launch are updated side by side, so a tensor that shares memory with one before it (layers with tied
// weights or a common bias) starts the next launch: updates of one element follow each other in the order of the list.
int launch_sgd(const SgdList &all, float lr, hipStream_t stream) {
    for (int t0 = 0; t0 < all.count;) {
        SgdList s;
        unsigned blocks = 0;
        int t = t0;
        for (; t < all.count; ++t) {
            if (!all.W[t] || !all.dW[t] || all.n[t] <= 0) CG_FAIL(CAPGNN_EINVAL, "sgd: NULL operand");
            bool shared = false;
            for (int u = 0; u < s.count && !shared; ++u)
                shared = overlap(all.W[t], all.n[t], s.W[u], s.n[u]) || overlap(all.W[t], all.n[t], s.dW[u], s.n[u]) ||
                         overlap(all.dW[t], all.n[t], s.W[u], s.n[u]);
            if (shared) break;
            s.W[s.count] = all.W[t]; s.dW[s.count] = all.dW[t]; s.n[s.count] = all.n[t];
            s.first[s.count++] = blocks;
            blocks += static_cast<unsigned>(std::min<int64_t>((all.n[t] + 255) / 256, 2048));
        }
        hipLaunchKernelGGL(sgd_kernel, dim3(blocks), dim3(256), 0, stream, s, lr);
        CG_HIP(hipGetLastError());
        t0 = t;
    }
    return CAPGNN_OK;
}

// ------------------------------------------------------------------ masked softmax / binary cross-entropy
// scratch layout (bytes): [0] normaliser (float); [256, LOSS_HEADER) partial counts of the mask (double); [LOSS_HEADER ..]
// per-workgroup partial sums of the loss (double).  All reductions have fixed summation orders.
constexpr int LOSS_PARTS = 512;
constexpr size_t LOSS_HEADER = 8192;

// threads: a power of two
__device__ __forceinline__ double block_sum(double c, double *red, int threads) {
    red[threadIdx.x] = c;
    __syncthreads();
    for (int s = threads / 2; s > 0; s >>= 1) {
        if (static_cast<int>(threadIdx.x) < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

__device__ __forceinline__ int nonzero_bytes(uint32_t w) {
    return ((w & 0xffu) != 0) + ((w & 0xff00u) != 0) + ((w & 0xff0000u) != 0) + ((w & 0xff000000u) != 0);
}

// nonzero bytes of [lo, hi), shared by `threads` threads; 16 at a time when the mask starts on a 16-byte boundary
__device__ __forceinline__ int count_range(const uint8_t *mask, int64_t lo, int64_t hi, int threads) {
    int cnt = 0;
    int64_t i = lo;
    if (reinterpret_cast<uintptr_t>(mask + lo) % 16 == 0) {
        const uint4 *m4 = reinterpret_cast<const uint4 *>(mask + lo);
        const int64_t n16 = (hi - lo) / 16;
        for (int64_t j = threadIdx.x; j < n16; j += threads) {
            const uint4 v = m4[j];
            cnt += nonzero_bytes(v.x) + nonzero_bytes(v.y) + nonzero_bytes(v.z) + nonzero_bytes(v.w);
        }
        i = lo + n16 * 16;
    }
    for (i += threadIdx.x; i < hi; i += threads) cnt += mask[i] ? 1 : 0;
    return cnt;
}

// part[b] = number of masked rows in workgroup b's contiguous slice (a multiple of 16 rows); bits (optional): one bit per row
__global__ __launch_bounds__(1024) void count_mask_kernel(int64_t n, const uint8_t *mask, double *part, uint16_t *bits) {
    __shared__ double red[1024];
    const int64_t per = ((n + gridDim.x - 1) / gridDim.x + 15) / 16 * 16;
    const int64_t lo = blockIdx.x * per < n ? blockIdx.x * per : n, hi = lo + per < n ? lo + per : n;
    if (bits)
        for (int64_t i = lo + 16 * static_cast<int64_t>(threadIdx.x); i < hi; i += 16 * 1024) {
            uint32_t m = 0;
            for (int j = 0; j < 16 && i + j < hi; ++j) m |= mask[i + j] ? 1u << j : 0u;
            bits[i / 16] = static_cast<uint16_t>(m);
        }
    const double c = block_sum(count_range(mask, lo, hi, 1024), red, 1024);
    if (threadIdx.x == 0) part[blockIdx.x] = c;
}

// norm_out[0] = max(sum of part, 1) * times, norm_out[1] = the sum itself
__global__ __launch_bounds__(LOSS_PARTS) void count_final_kernel(int parts, const double *part, float times, float *norm_out) {
    __shared__ double red[LOSS_PARTS];
    const double c = block_sum(static_cast<int>(threadIdx.x) < parts ? part[threadIdx.x] : 0.0, red, LOSS_PARTS);
    if (threadIdx.x == 0) {
        norm_out[0] = (c > 0.0 ? static_cast<float>(c) : 1.f) * times;
        norm_out[1] = static_cast<float>(c);
    }
}

// Up to this many rows one workgroup counts the mask (the two-level form costs a second launch) ...
constexpr int64_t COUNT_SMALL_N = int64_t(1) << 18;
__global__ __launch_bounds__(1024) void count_small_kernel(int64_t n, const uint8_t *mask, float times, float *norm_out) {
    __shared__ double red[1024];
    const double c = block_sum(count_range(mask, 0, n, 1024), red, 1024);
    if (threadIdx.x == 0) norm_out[0] = (c > 0.0 ? static_cast<float>(c) : 1.f) * times;
}
// ... and up to this many every workgroup of the loss kernel counts it for itself: at most 64 bytes per thread, out of
// the L2, instead of a launch of its own (3-4 us).
constexpr int64_t COUNT_INLINE_N = int64_t(1) << 14;

// Workgroups of the loss kernel that a compute unit holds at once: the grid is that many on every unit and no more, since all
// of them walk equally many rows (2048 workgroups where 1792 fit: 980 k rows x 47 classes 240 us, 72 us for 306 k rows).
template <bool BCE> constexpr int LOSS_WG_PER_CU = BCE ? 5 : 8;

// A group of lpr lanes (a power of two, 4..64, about a quarter of the classes) per row, so that narrow class counts
// still keep 64/lpr rows in flight per wave; the lanes of a group stride over the classes.
static int loss_lanes_per_row_host(int C) {
    int lpr = 4;
    while (lpr < 64 && lpr * 4 < C) lpr *= 2;
    return lpr;
}

struct LossArgs {
    int64_t n;
    int C, lpr;
    const float *Z; int64_t ldz;
    const int32_t *labels;              // softmax: class of every row
    const uint8_t *targets; int64_t ldt;   // binary: 0/1 matrix
    const uint8_t *mask;
    float norm_val; const float *norm_dev;  // the normaliser, or where it is
    float norm_times;                   // > 0: the normaliser is the mask's count times this, counted by every workgroup
    double *part;                       // [gridDim.x] sums of the row losses
    float *norm_out;                    // where workgroup 0 leaves a normaliser counted here, or null
    char *dZ; int64_t lddz; int dz_bf16;
    const float *rscale;                // dZ rows are stored times this, or null
    float *copy;                        // dense [n x C] copy of the logits, or null
    float *colpart;                     // [gridDim.x][C] column sums of dZ (not scaled), or null; C <= 4 * lpr
};

// One lane group per row, rows strided over the grid; the next row's logits are on their way while a row is worked on.  A lane
// keeps up to four logits (classes l, l + lpr, ...), which covers every C <= 4 * lpr (all C <= 256); beyond that the row is
// read again from the L1.  One exponential per class.  Softmax: p_k = e_k / s.  Binary: the element's loss in the form
// max(z,0) - z*y + log(1 + exp(-|z|)), which neither overflows nor cancels, and its derivative s(z) - y.
// The kernel also sums the row losses and, for the layer's bias gradient, the columns of dZ: what were passes of their own
// over the rows' terms and over dZ (a 4096-vertex epoch: five launches, 35 us, now two).
template <bool BCE>
__global__ __launch_bounds__(256, LOSS_WG_PER_CU<BCE>) void loss_kernel(LossArgs a) {
    constexpr int KEEP = 4;
    __shared__ double red[256];
    __shared__ float cred[4][4 * 64];
    const int lpr = a.lpr, C = a.C;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l = lane % lpr;
    const int64_t per = static_cast<int64_t>(gridDim.x) * 4 * (64 / lpr);
    int64_t row = (static_cast<int64_t>(blockIdx.x) * 4 + wave) * (64 / lpr) + lane / lpr;
    const bool kept = C <= KEEP * lpr;
    float zn[KEEP], tn[KEEP];
    bool on_n = false;
    int y_n = 0;
    auto fetch = [&](int64_t r) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < KEEP; ++j) {
            const int k = l + j * lpr;
            zn[j] = r < a.n && k < C ? a.Z[r * a.ldz + k] : -INFINITY;
            if constexpr (BCE) tn[j] = r < a.n && k < C && a.targets[r * a.ldt + k] ? 1.f : 0.f;
        }
        on_n = r < a.n && (!a.mask || a.mask[r]);
        if constexpr (!BCE) y_n = r < a.n ? a.labels[r] : 0;
    };
    fetch(row);
    float norm = a.norm_val;
    if (a.norm_times > 0.f) {           // uniform over the grid
        const double c = block_sum(count_range(a.mask, 0, a.n, 256), red, 256);
        norm = (c > 0.0 ? static_cast<float>(c) : 1.f) * a.norm_times;
        if (a.norm_out && blockIdx.x == 0 && threadIdx.x == 0) a.norm_out[0] = norm;
        __syncthreads();
    } else if (a.norm_dev) {
        norm = a.norm_dev[0];
    }
    const float inv = 1.f / norm;
    double loss = 0.0;
    float csum[KEEP] = {0.f, 0.f, 0.f, 0.f};
    for (; __any(row < a.n); row += per) {
        float z[KEEP], t[KEEP];
#pragma unroll
        for (int j = 0; j < KEEP; ++j) {
            z[j] = zn[j];
            if constexpr (BCE) t[j] = tn[j];
        }
        const bool in = row < a.n, on = on_n;
        int y = y_n;
        fetch(row + per);
        const float *zr = a.Z + row * a.ldz;
        if (in && a.copy) {
#pragma unroll
            for (int j = 0; j < KEEP; ++j)
                if (l + j * lpr < C) a.copy[row * C + l + j * lpr] = z[j];
            if (!kept) for (int k = l + KEEP * lpr; k < C; k += lpr) a.copy[row * C + k] = zr[k];
        }
        float d[KEEP] = {0.f, 0.f, 0.f, 0.f};
        float term = 0.f, m = -INFINITY, inv_s = 0.f;
        if constexpr (BCE) {
            if (on) {
#pragma unroll
                for (int j = 0; j < KEEP; ++j) {
                    if (l + j * lpr >= C) continue;
                    const float e = expf(-fabsf(z[j]));
                    term += fmaxf(z[j], 0.f) - z[j] * t[j] + log1pf(e);
                    d[j] = ((z[j] >= 0.f ? 1.f / (1.f + e) : e / (1.f + e)) - t[j]) * inv;
                }
                if (!kept)
                    for (int k = l + KEEP * lpr; k < C; k += lpr) {
                        const float zk = zr[k], yk = a.targets[row * a.ldt + k] ? 1.f : 0.f;
                        term += fmaxf(zk, 0.f) - zk * yk + log1pf(expf(-fabsf(zk)));
                    }
            }
            for (int off = lpr >> 1; off > 0; off >>= 1) term += __shfl_xor(term, off);
        } else {
            y = y < 0 ? 0 : (y >= C ? C - 1 : y);
            m = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
            if (in && !kept) for (int k = l + KEEP * lpr; k < C; k += lpr) m = fmaxf(m, zr[k]);
            for (int off = lpr >> 1; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
            float er[KEEP], s = 0.f, zy = 0.f;
#pragma unroll
            for (int j = 0; j < KEEP; ++j) {
                const int k = l + j * lpr;
                er[j] = in && k < C ? expf(z[j] - m) : 0.f;
                s += er[j];
                if (k == y) zy = z[j];
            }
            if (in && !kept)
                for (int k = l + KEEP * lpr; k < C; k += lpr) {
                    s += expf(zr[k] - m);
                    if (k == y) zy = zr[k];
                }
            for (int off = lpr >> 1; off > 0; off >>= 1) { s += __shfl_xor(s, off); zy += __shfl_xor(zy, off); }
            inv_s = 1.f / s;
            if (on) {
                term = m + logf(s) - zy;
#pragma unroll
                for (int j = 0; j < KEEP; ++j) d[j] = (er[j] * inv_s - (l + j * lpr == y ? 1.f : 0.f)) * inv;
            }
        }
        if (on && l == 0) loss += static_cast<double>(term);
        if (in && a.dZ) {
            const float rs = a.rscale ? a.rscale[row] : 1.f;
#pragma unroll
            for (int j = 0; j < KEEP; ++j) {
                const int k = l + j * lpr;
                if (k < C) st_elem(a.dZ, row * a.lddz + k, d[j] * rs, a.dz_bf16);
            }
            if (!kept)
                for (int k = l + KEEP * lpr; k < C; k += lpr) {
                    float g = 0.f;
                    if (on) {
                        if constexpr (BCE) {
                            const float zk = zr[k], yk = a.targets[row * a.ldt + k] ? 1.f : 0.f, e = expf(-fabsf(zk));
                            g = ((zk >= 0.f ? 1.f / (1.f + e) : e / (1.f + e)) - yk) * inv;
                        } else {
                            g = (expf(zr[k] - m) * inv_s - (k == y ? 1.f : 0.f)) * inv;
                        }
                    }
                    st_elem(a.dZ, row * a.lddz + k, g * rs, a.dz_bf16);
                }
        }
#pragma unroll
        for (int j = 0; j < KEEP; ++j) csum[j] += in ? d[j] : 0.f;
    }
    const double c = block_sum(loss, red, 256);
    if (threadIdx.x == 0) a.part[blockIdx.x] = c;
    if (!a.colpart) return;
    for (int off = lpr; off < 64; off <<= 1)
#pragma unroll
        for (int j = 0; j < KEEP; ++j) csum[j] += __shfl_xor(csum[j], off);
    if (lane < lpr)
#pragma unroll
        for (int j = 0; j < KEEP; ++j) cred[wave][l + j * lpr] = csum[j];
    __syncthreads();
    for (int k = threadIdx.x; k < C; k += 256)
        a.colpart[static_cast<int64_t>(blockIdx.x) * C + k] = (cred[0][k] + cred[1][k]) + (cred[2][k] + cred[3][k]);
}

// workgroup 0: loss = sum of part / normaliser; the others (when there is a bias gradient): 32 columns each, as dbias_final_kernel
__global__ __launch_bounds__(1024) void loss_final_kernel(int parts, const double *part, float norm_val, const float *norm_dev,
                                                          float *loss_out, const float *colpart, int C, float *dbias) {
    __shared__ double red[1024];
    if (blockIdx.x == 0) {
        double c = 0.0;
        for (int b = threadIdx.x; b < parts; b += 1024) c += part[b];
        c = block_sum(c, red, 1024);
        if (threadIdx.x == 0) loss_out[0] = static_cast<float>(c / (norm_dev ? static_cast<double>(norm_dev[0]) : static_cast<double>(norm_val)));
        return;
    }
    column_sums(blockIdx.x - 1, parts, C, colpart, dbias, red);
}

// The end of an epoch in one launch: sums over the splits of every weight gradient (as gemm_reduce_kernel adds them), over the
// loss's workgroups, and the SGD step, which the thread that has a sum applies.  They were a launch each (a 4096-vertex epoch: four
// of fifteen, 3-4 us apiece; 81 -> 72 us with the gathers of all layers in one launch).  A workgroup takes 4 x 32 sums with eight
// threads each, or 32 columns of the loss's with 32 threads each, or the loss, or 4096 elements of an update.
constexpr int FINISH_UPDATES = 4096;
__global__ __launch_bounds__(1024) void epoch_finish_kernel(FinishList list, float lr) {
    __shared__ double red[1024];
    int i = 0;
    while (i + 1 < list.count && blockIdx.x >= list.task[i + 1].first) ++i;
    const FinishTask &t = list.task[i];
    const int64_t b = blockIdx.x - t.first;
    if (t.kind == FinishTask::SUM || t.kind == FinishTask::COLUMNS) {
        const int tx = threadIdx.x & 31, ty = (threadIdx.x >> 5) & 7, quarter = threadIdx.x >> 8;
        const int64_t e = b * 128 + quarter * 32 + tx;
        const float *part = static_cast<const float *>(t.part);
        double v = 0.0;
        if (e < t.n && t.kind == FinishTask::SUM) {
            float f = 0.f;
            int z = ty;
            for (; z + 56 < t.S; z += 64) {
                float q[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) q[u] = part[static_cast<int64_t>(z + 8 * u) * t.n + e];
#pragma unroll
                for (int u = 0; u < 8; ++u) f += q[u];
            }
            for (; z < t.S; z += 8) f += part[static_cast<int64_t>(z) * t.n + e];
            v = f;
        } else if (e < t.n) {
            for (int z = ty; z < t.S; z += 8) v += static_cast<double>(part[static_cast<int64_t>(z) * t.n + e]);
        }
        double *r = red + quarter * 256;
        r[ty * 32 + tx] = v;
        __syncthreads();
        if (ty != 0 || e >= t.n) return;
        float sum;
        if (t.kind == FinishTask::SUM) {
            sum = 0.f;
            for (int y = 0; y < 8; ++y) sum += static_cast<float>(r[y * 32 + tx]);
        } else {
            v = 0.0;
            for (int y = 0; y < 8; ++y) v += r[y * 32 + tx];
            sum = static_cast<float>(v);
        }
        t.out[e] = sum;
        if (t.W) t.W[e] = t.W[e] - lr * sum;
    } else if (t.kind == FinishTask::LOSS_COLUMNS) {
        column_sums(static_cast<unsigned>(b), t.S, static_cast<int>(t.n), static_cast<const float *>(t.part), t.out, red);
        const int64_t e = b * 32 + threadIdx.x;
        if (threadIdx.x < 32 && e < t.n && t.W) t.W[e] = t.W[e] - lr * t.out[e];      // (the thread that wrote it)
    } else if (t.kind == FinishTask::LOSS) {
        const double *part = static_cast<const double *>(t.part);
        double c = 0.0;
        for (int k = threadIdx.x; k < t.S; k += 1024) c += part[k];
        c = block_sum(c, red, 1024);
        if (threadIdx.x == 0) {
            const float loss = static_cast<float>(c / (t.norm_dev ? static_cast<double>(t.norm_dev[0]) : static_cast<double>(t.norm_val)));
            t.out[0] = loss;
            if (t.out2) t.out2[0] = loss;
        }
    } else {
        const float *dW = static_cast<const float *>(t.part);
        for (int64_t e = b * FINISH_UPDATES + threadIdx.x; e < t.n && e < (b + 1) * FINISH_UPDATES; e += 1024) t.W[e] = t.W[e] - lr * dW[e];
    }
}

static int64_t finish_blocks(const FinishTask &t) {
    switch (t.kind) {
        case FinishTask::SUM: case FinishTask::COLUMNS: return (t.n + 127) / 128;
        case FinishTask::LOSS_COLUMNS: return (t.n + 31) / 32;
        case FinishTask::LOSS: return 1;
        default: return (t.n + FINISH_UPDATES - 1) / FINISH_UPDATES;
    }
}

static int launch_tasks(FinishList *l, float lr, hipStream_t stream) {
    int64_t blocks = 0;
    for (int i = 0; i < l->count; ++i) {
        l->task[i].first = static_cast<unsigned>(blocks);
        blocks += finish_blocks(l->task[i]);
    }
    if (blocks == 0) return CAPGNN_OK;
    hipLaunchKernelGGL(epoch_finish_kernel, dim3(static_cast<unsigned>(blocks)), dim3(1024), 0, stream, *l, lr);
    CG_HIP(hipGetLastError());
    return CAPGNN_OK;
}

// Tasks of one launch run side by side.  Where tensors share memory (tied weights, a common bias, one buffer for two gradients) the
// sums are written by one launch each, in their order, and launch_sgd follows, which keeps to the order of its own list.
int launch_finish(FinishList *list, const SgdList *sgd, float lr, hipStream_t stream) {
    FinishList l = *list;
    bool apart = true;
    if (lr != 0.f && sgd) {
        for (int u = 0; u < sgd->count; ++u) {
            if (!sgd->W[u] || !sgd->dW[u] || sgd->n[u] <= 0) CG_FAIL(CAPGNN_EINVAL, "sgd: NULL operand");
            FinishTask *own = nullptr;
            for (int i = 0; i < list->count && !own; ++i)
                if (l.task[i].kind != FinishTask::LOSS && l.task[i].out == sgd->dW[u] && l.task[i].n == sgd->n[u] && !l.task[i].W) own = &l.task[i];
            if (own) { own->W = sgd->W[u]; continue; }
            if (l.full()) { apart = false; break; }
            FinishTask t{};
            t.kind = FinishTask::UPDATE; t.n = sgd->n[u]; t.part = sgd->dW[u]; t.W = sgd->W[u];
            l.task[l.count++] = t;
        }
    }
    // the memory a task writes, against everything that another reads or writes of the caller's
    auto spans = [](const FinishTask &t, const float *(&p)[4], int64_t (&n)[4]) {
        p[0] = t.out; n[0] = t.out ? (t.kind == FinishTask::LOSS ? 1 : t.n) : 0;
        p[1] = t.W; n[1] = t.W ? t.n : 0;
        p[2] = t.out2; n[2] = t.out2 ? 1 : 0;
        p[3] = t.kind == FinishTask::UPDATE ? static_cast<const float *>(t.part) : nullptr; n[3] = p[3] ? t.n : 0;
    };
    for (int i = 0; i < l.count && apart; ++i) {
        const float *p[4]; int64_t n[4];
        spans(l.task[i], p, n);
        for (int j = 0; j <= i && apart; ++j) {
            const float *q[4]; int64_t m[4];
            spans(l.task[j], q, m);
            for (int x = 0; x < 4; ++x)
                for (int y = 0; y < 4; ++y)
                    if ((x != 3 || y != 3) && (i != j || x < y) && n[x] && m[y] && overlap(p[x], n[x], q[y], m[y])) apart = false;
        }
    }
    if (apart) return launch_tasks(&l, lr, stream);
    for (int i = 0; i < list->count; ++i) {
        FinishList one;
        one.task[one.count++] = list->task[i];
        CG_TRY(launch_tasks(&one, lr, stream));
    }
    return lr != 0.f && sgd ? launch_sgd(*sgd, lr, stream) : CAPGNN_OK;
}

static int loss_blocks(int64_t n, int C, bool bce) {
    const int64_t rows = 4 * (64 / loss_lanes_per_row_host(C));
    return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((n + rows - 1) / rows, NUM_CU * (bce ? LOSS_WG_PER_CU<true> : LOSS_WG_PER_CU<false>))));
}

// a: everything but the normaliser and `part`.  times: what the mask's count is multiplied with for the normaliser.
// colpart (loss_colpart_bytes) and dbias: also the layer's bias gradient.
// bits (with a mask): one bit per row of the mask is left there, and the number of set ones in norm_dev[1].
static int loss_launch(LossArgs a, bool bce, double loss_norm, float times, float *loss_dev, void *ws, float *colpart, float *dbias,
                       hipStream_t st, uint16_t *bits = nullptr, FinishList *later = nullptr) {
    float *norm_dev = static_cast<float *>(ws);
    double *counts = reinterpret_cast<double *>(static_cast<char *>(ws) + 256);
    a.part = reinterpret_cast<double *>(static_cast<char *>(ws) + LOSS_HEADER);
    a.lpr = loss_lanes_per_row_host(a.C);
    a.norm_val = 1.f; a.norm_dev = nullptr; a.norm_times = 0.f; a.norm_out = nullptr;
    if (a.mask && (bits || (loss_norm <= 0.0 && a.n > COUNT_SMALL_N))) {
        const int parts = static_cast<int>(std::min<int64_t>((a.n + 4095) / 4096, LOSS_PARTS));
        hipLaunchKernelGGL(count_mask_kernel, dim3(parts), dim3(1024), 0, st, a.n, a.mask, counts, bits);
        hipLaunchKernelGGL(count_final_kernel, dim3(1), dim3(LOSS_PARTS), 0, st, parts, counts, times, norm_dev);
        if (loss_norm <= 0.0) a.norm_dev = norm_dev;
    }
    if (loss_norm > 0.0) {
        a.norm_val = static_cast<float>(loss_norm);
    } else if (!a.mask) {
        a.norm_val = static_cast<float>(a.n) * times;
    } else if (a.norm_dev) {
        // counted above
    } else if (a.n <= COUNT_INLINE_N) {
        a.norm_times = times;
        a.norm_out = norm_dev;
    } else {
        a.norm_dev = norm_dev;
        hipLaunchKernelGGL(count_small_kernel, dim3(1), dim3(1024), 0, st, a.n, a.mask, times, norm_dev);
    }
    const int blocks = loss_blocks(a.n, a.C, bce);
    a.colpart = dbias ? colpart : nullptr;
    if (bce) hipLaunchKernelGGL(loss_kernel<true>, dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(loss_kernel<false>, dim3(blocks), dim3(256), 0, st, a);
    if (later && later->count + 2 <= FinishList::MOST) {
        FinishTask t{};
        t.kind = FinishTask::LOSS; t.S = blocks; t.n = 1; t.part = a.part; t.out = loss_dev;
        t.norm_val = a.norm_val; t.norm_dev = (a.norm_dev || a.norm_out) ? norm_dev : nullptr;
        later->task[later->count++] = t;
        if (dbias) {
            t = FinishTask{};
            t.kind = FinishTask::LOSS_COLUMNS; t.S = blocks; t.n = a.C; t.part = a.colpart; t.out = dbias;
            later->task[later->count++] = t;
        }
        CG_HIP(hipGetLastError());
        return CAPGNN_OK;
    }
    hipLaunchKernelGGL(loss_final_kernel, dim3(1 + (dbias ? (a.C + 31) / 32 : 0)), dim3(1024), 0, st, blocks, a.part, a.norm_val,
                       (a.norm_dev || a.norm_out) ? norm_dev : nullptr, loss_dev, a.colpart, a.C, dbias);
    CG_HIP(hipGetLastError());
    return CAPGNN_OK;
}

}  // namespace capgnn

using namespace capgnn;

extern "C" size_t capgnn_loss_workspace_bytes(int64_t n) {
    return align_up(LOSS_HEADER + static_cast<size_t>(n > 0 ? n : 1) * sizeof(float), 256);
}

extern "C" int capgnn_sigmoid_bce(int64_t n, int C, const float *Z, int64_t ldz, const uint8_t *targets, int64_t ldt,
                                  const uint8_t *mask, double loss_norm, float *loss_dev, void *dZ, int64_t lddz,
                                  int dz_dtype, void *ws, size_t ws_bytes, void *stream) {
    if (dz_dtype != CAPGNN_F32 && dz_dtype != CAPGNN_BF16) CG_FAIL(CAPGNN_EINVAL, "sigmoid_bce: unknown dz_dtype");
    if (n < 0 || C <= 0) CG_FAIL(CAPGNN_EINVAL, "sigmoid_bce: bad sizes");
    if (n == 0) return CAPGNN_OK;
    if (!Z || !targets || !loss_dev) CG_FAIL(CAPGNN_EINVAL, "sigmoid_bce: NULL operand");
    if (ldz < C || ldt < C || (dZ && lddz < C)) CG_FAIL(CAPGNN_EINVAL, "sigmoid_bce: leading dimension smaller than C");
    if (!ws || ws_bytes < capgnn_loss_workspace_bytes(n)) CG_FAIL(CAPGNN_ENOMEM, "sigmoid_bce: workspace too small");
    LossArgs a{};
    a.n = n; a.C = C; a.Z = Z; a.ldz = ldz; a.targets = targets; a.ldt = ldt; a.mask = mask;
    a.dZ = static_cast<char *>(dZ); a.lddz = lddz; a.dz_bf16 = dz_dtype == CAPGNN_BF16;
    return loss_launch(a, true, loss_norm, static_cast<float>(C), loss_dev, ws, nullptr, nullptr, static_cast<hipStream_t>(stream));
}

// everything capgnn_softmax_ce does after its argument checks; `ws` holds capgnn_loss_workspace_bytes(n) bytes
static int softmax_ce_launch(int64_t n, int C, const float *Z, int64_t ldz, const int32_t *labels, const uint8_t *mask,
                             double loss_norm, float *loss_dev, void *dZ, int64_t lddz, int dz_dtype, void *ws, hipStream_t st) {
    LossArgs a{};
    a.n = n; a.C = C; a.Z = Z; a.ldz = ldz; a.labels = labels; a.mask = mask;
    a.dZ = static_cast<char *>(dZ); a.lddz = lddz; a.dz_bf16 = dz_dtype == CAPGNN_BF16;
    return loss_launch(a, false, loss_norm, 1.f, loss_dev, ws, nullptr, nullptr, st);
}

static int softmax_ce_check(int64_t n, int C, const float *Z, int64_t ldz, const int32_t *labels, float *loss_dev,
                            const void *dZ, int64_t lddz, int dz_dtype) {
    if (dz_dtype != CAPGNN_F32 && dz_dtype != CAPGNN_BF16) CG_FAIL(CAPGNN_EINVAL, "softmax_ce: unknown dz_dtype");
    if (n < 0 || C <= 0) CG_FAIL(CAPGNN_EINVAL, "softmax_ce: bad sizes");
    if (n == 0) return CAPGNN_OK;
    if (!Z || !labels || !loss_dev) CG_FAIL(CAPGNN_EINVAL, "softmax_ce: NULL operand");
    if (ldz < C || (dZ && lddz < C)) CG_FAIL(CAPGNN_EINVAL, "softmax_ce: leading dimension smaller than C");
    return CAPGNN_OK;
}

extern "C" int capgnn_softmax_ce(int64_t n, int C, const float *Z, int64_t ldz, const int32_t *labels,
                                 const uint8_t *mask, double loss_norm, float *loss_dev, void *dZ, int64_t lddz,
                                 int dz_dtype, void *ws, size_t ws_bytes, void *stream) {
    CG_TRY(softmax_ce_check(n, C, Z, ldz, labels, loss_dev, dZ, lddz, dz_dtype));
    if (n == 0) return CAPGNN_OK;
    if (!ws || ws_bytes < capgnn_loss_workspace_bytes(n)) CG_FAIL(CAPGNN_ENOMEM, "softmax_ce: workspace too small");
    return softmax_ce_launch(n, C, Z, ldz, labels, mask, loss_norm, loss_dev, dZ, lddz, dz_dtype, ws,
                             static_cast<hipStream_t>(stream));
}

size_t capgnn::loss_epoch_ws_bytes(int64_t n, int C) {
    return capgnn_loss_workspace_bytes(n) + align_up(static_cast<size_t>(loss_blocks(n, C, false)) * C * sizeof(float), 256) +
           align_up(static_cast<size_t>(n > 0 ? (n + 31) / 32 : 0) * sizeof(uint32_t), 256);
}

bool capgnn::loss_sums_columns(int C) { return C <= 4 * loss_lanes_per_row_host(C); }

// The loss of an epoch (labels or targets): also writes the logits as a dense [n x C] matrix to `copy`, sums the columns of dZ
// into dbias, and stores the rows of dZ times row_scale (each may be NULL).  live (with a mask): where the rows are that have a
// gradient, in `ws`.
int capgnn::loss_epoch(int64_t n, int C, const float *Z, int64_t ldz, const int32_t *labels, const uint8_t *targets, int64_t ldt,
                       const uint8_t *mask, double loss_norm, float *loss_dev, void *dZ, int64_t lddz, int dz_dtype, float *copy,
                       float *dbias, const float *row_scale, LiveRows *live, void *ws, size_t ws_bytes, hipStream_t st, FinishList *later) {
    CG_TRY(softmax_ce_check(n, C, Z, ldz, targets ? reinterpret_cast<const int32_t *>(targets) : labels, loss_dev, dZ, lddz, dz_dtype));
    if (n == 0) return CAPGNN_OK;
    if (targets && ldt < C) CG_FAIL(CAPGNN_EINVAL, "loss: ldt smaller than the number of classes");
    if (dbias && !loss_sums_columns(C)) CG_FAIL(CAPGNN_EINVAL, "loss: too many classes for the column sums");
    if (!ws || ws_bytes < loss_epoch_ws_bytes(n, C)) CG_FAIL(CAPGNN_ENOMEM, "loss: workspace too small");
    LossArgs a{};
    a.n = n; a.C = C; a.Z = Z; a.ldz = ldz; a.labels = labels; a.targets = targets; a.ldt = ldt; a.mask = mask;
    a.dZ = static_cast<char *>(dZ); a.lddz = lddz; a.dz_bf16 = dz_dtype == CAPGNN_BF16; a.copy = copy; a.rscale = row_scale;
    char *colpart = static_cast<char *>(ws) + capgnn_loss_workspace_bytes(n);
    uint16_t *bits = nullptr;
    if (live && mask) {
        bits = reinterpret_cast<uint16_t *>(colpart + align_up(static_cast<size_t>(loss_blocks(n, C, false)) * C * sizeof(float), 256));
        live->bits = reinterpret_cast<const uint32_t *>(bits);
        live->count = static_cast<const float *>(ws) + 1;
    }
    return loss_launch(a, targets != nullptr, loss_norm, targets ? static_cast<float>(C) : 1.f, loss_dev, ws,
                       reinterpret_cast<float *>(colpart), dbias, st, bits, later);
}

// ------------------------------------------------------------------ the same loss without any allocation by anyone
// The scratch of capgnn_softmax_ce (normaliser, per-workgroup partial sums) for up to
// CAPGNN_LOSS_STATIC_MAX_ROWS rows, as a device array that is part of the library image: every GPU the library
// runs on holds its own copy until the process ends.  Host code never uses the array's name as an address: the
// address on the current device is asked for once per device and kept.
static __device__ __align__(256) unsigned char scratch[LOSS_HEADER + static_cast<size_t>(CAPGNN_LOSS_STATIC_MAX_ROWS) * sizeof(float)];

constexpr int MAX_DEVICES = 64;
static void *g_scratch_ptr[MAX_DEVICES];
static std::mutex g_scratch_mutex;

// device address of `scratch` on the current device (looked up on the first call on that device)
static int static_scratch(void **out) {
    int dev = -1;
    CG_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) CG_FAIL(CAPGNN_EUNSUPPORTED, "softmax_ce_static: device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        CG_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) CG_FAIL(CAPGNN_EHIP, "softmax_ce_static: the scratch array has no address on device %d", dev);
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return CAPGNN_OK;
}

extern "C" int capgnn_softmax_ce_static(int64_t n, int C, const float *Z, int64_t ldz, const int32_t *labels,
                                        const uint8_t *mask, double loss_norm, float *loss_dev, void *dZ, int64_t lddz,
                                        int dz_dtype, void *stream) {
    CG_TRY(softmax_ce_check(n, C, Z, ldz, labels, loss_dev, dZ, lddz, dz_dtype));
    if (n > CAPGNN_LOSS_STATIC_MAX_ROWS)
        CG_FAIL(CAPGNN_ENOMEM, "softmax_ce_static: %lld rows, the built-in scratch holds %d; use capgnn_softmax_ce with a workspace",
                static_cast<long long>(n), CAPGNN_LOSS_STATIC_MAX_ROWS);
    if (n == 0) return CAPGNN_OK;
    void *ws = nullptr;
    CG_TRY(static_scratch(&ws));
    // nothing in the scratch has to start at zero: the normaliser and the partial sums are all written before they are read, so what an earlier (larger) call left behind is never seen
    return softmax_ce_launch(n, C, Z, ldz, labels, mask, loss_norm, loss_dev, dZ, lddz, dz_dtype, ws,
                             static_cast<hipStream_t>(stream));
}
