// Normalised sparse aggregation Y = A_hat X (and, over the CSC, dX = A_hat^T dY) for gfx950.
//
// LPR lanes (a power of two, as many as a feature row has 16-byte vectors, at most a whole wave) cover one feature row, so a
// wave gathers the rows of 64 / LPR entries with one instruction.  Short output rows are given to one lane group each, so
// that a wave works on 64 / LPR of them at a time; longer ones, and pieces of very long ones, to a whole wave, whose groups
// share the entries.  Either way every lane has eight feature-row loads in flight.  The column indices are read one per
// lane, together with the per-entry weight (edge_val * in_scale[col], formed at graph creation), and handed from lane to
// lane.  The pieces of a cut row are summed in a fixed order by a second kernel: results are reproducible run to run.
#include "common.h"

#include <algorithm>

namespace capgnn {

struct SpmmArgs {
    const int32_t *idx;
    const float *out_scale;
    const float *wt;          // per-entry weights, or null: every weight is 1
    const RowItem *items;     // [n_items]
    int64_t n_items, n_pieces;   // the first n_pieces items are pieces of cut rows: raw sums to `part`
    int64_t n_wave;              // the first n_wave items (pieces among them) are given a whole wave each
    const char *X;
    int64_t ldx_bytes;
    char *Y;
    int64_t ldy_bytes;
    int F;        // valid elements per row
    int F_lim;    // elements covered by loads (F rounded up to the vector width)
    const float *bias;
    int relu;
    int acc_rows;             // output rows below this one are added to what Y holds
    const char *mask;         // zero where mask <= 0 (storage type of Y), or null
    int64_t ldm_bytes;
    LiveRows live;            // rows of X that may differ from zero (LIVE kernels)
    int64_t n_in;
    float *part;              // fp32 partial sums [n_pieces][ldp]
    int64_t ldp;
};

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);                                   // round to nearest even
    return u >> 16;
}

template <bool BF16, int E>
__device__ __forceinline__ void load_elems(const char *p, float (&x)[E]) {
    if constexpr (!BF16 && E == 4) {
        float4 v = *reinterpret_cast<const float4 *>(p);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else if constexpr (!BF16 && E == 1) {
        x[0] = *reinterpret_cast<const float *>(p);
    } else if constexpr (BF16 && E == 8) {
        uint4 v = *reinterpret_cast<const uint4 *>(p);
        x[0] = __uint_as_float(v.x << 16); x[1] = __uint_as_float(v.x & 0xffff0000u);
        x[2] = __uint_as_float(v.y << 16); x[3] = __uint_as_float(v.y & 0xffff0000u);
        x[4] = __uint_as_float(v.z << 16); x[5] = __uint_as_float(v.z & 0xffff0000u);
        x[6] = __uint_as_float(v.w << 16); x[7] = __uint_as_float(v.w & 0xffff0000u);
    } else {
        static_assert(BF16 && E == 1, "unsupported element packing");
        x[0] = bf16_bits_to_f32(*reinterpret_cast<const uint16_t *>(p));
    }
}

// The same elements kept as loaded (packed bf16 stay packed: half the registers while several loads are in flight)
// and widened only when they are consumed.
template <bool BF16, int E> struct RawVec { float v[E]; };
template <> struct RawVec<true, 8> { uint4 v; };
template <> struct RawVec<true, 1> { uint16_t v; };

template <bool BF16, int E>
__device__ __forceinline__ void load_raw(const char *p, RawVec<BF16, E> &r) {
    if constexpr (BF16 && E == 8) r.v = *reinterpret_cast<const uint4 *>(p);
    else if constexpr (BF16 && E == 1) r.v = *reinterpret_cast<const uint16_t *>(p);
    else load_elems<BF16, E>(p, r.v);
}

template <bool BF16, int E>
__device__ __forceinline__ void zero_raw(RawVec<BF16, E> &r) {
    if constexpr (BF16 && E == 8) r.v = make_uint4(0u, 0u, 0u, 0u);
    else if constexpr (BF16 && E == 1) r.v = 0;
    else {
#pragma unroll
        for (int j = 0; j < E; ++j) r.v[j] = 0.f;
    }
}

// acc += w * r (W), or acc += r
template <bool BF16, bool W, int E>
__device__ __forceinline__ void fma_raw(float w, const RawVec<BF16, E> &r, float (&acc)[E]) {
    auto add = [w](float x, float &s) { s = W ? fmaf(w, x, s) : s + x; };
    if constexpr (BF16 && E == 8) {
        const uint32_t u[4] = {r.v.x, r.v.y, r.v.z, r.v.w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            add(__uint_as_float(u[d] << 16), acc[2 * d]);
            add(__uint_as_float(u[d] & 0xffff0000u), acc[2 * d + 1]);
        }
    } else if constexpr (BF16 && E == 1) {
        add(bf16_bits_to_f32(r.v), acc[0]);
    } else {
#pragma unroll
        for (int j = 0; j < E; ++j) add(r.v[j], acc[j]);
    }
}

template <bool BF16>
__device__ __forceinline__ float load_one(const char *p) {
    if constexpr (BF16) return bf16_bits_to_f32(*reinterpret_cast<const uint16_t *>(p));
    else return *reinterpret_cast<const float *>(p);
}

template <bool BF16>
__device__ __forceinline__ void store_one(char *p, float v) {
    if constexpr (BF16) *reinterpret_cast<uint16_t *>(p) = static_cast<uint16_t>(f32_to_bf16_bits(v));
    else *reinterpret_cast<float *>(p) = v;
}

template <bool BF16, int E>
__device__ __forceinline__ void store_elems(char *p, const float (&x)[E]) {
    if constexpr (!BF16 && E == 4) {
        *reinterpret_cast<float4 *>(p) = make_float4(x[0], x[1], x[2], x[3]);
    } else if constexpr (!BF16 && E == 8) {
        reinterpret_cast<float4 *>(p)[0] = make_float4(x[0], x[1], x[2], x[3]);
        reinterpret_cast<float4 *>(p)[1] = make_float4(x[4], x[5], x[6], x[7]);
    } else if constexpr (BF16 && E == 8) {
        uint4 v;
        v.x = f32_to_bf16_bits(x[0]) | (f32_to_bf16_bits(x[1]) << 16);
        v.y = f32_to_bf16_bits(x[2]) | (f32_to_bf16_bits(x[3]) << 16);
        v.z = f32_to_bf16_bits(x[4]) | (f32_to_bf16_bits(x[5]) << 16);
        v.w = f32_to_bf16_bits(x[6]) | (f32_to_bf16_bits(x[7]) << 16);
        *reinterpret_cast<uint4 *>(p) = v;
    } else if constexpr (BF16 && E == 4) {      // float operand, bf16 result: four elements per lane
        uint2 v;
        v.x = f32_to_bf16_bits(x[0]) | (f32_to_bf16_bits(x[1]) << 16);
        v.y = f32_to_bf16_bits(x[2]) | (f32_to_bf16_bits(x[3]) << 16);
        *reinterpret_cast<uint2 *>(p) = v;
    } else {
        static_assert(E == 1, "unsupported element packing");
        store_one<BF16>(p, x[0]);
    }
}

// Adds, for the entries [e, end) of one output row, weight * X[source, lane's features] to acc.
//   WAVE   the row belongs to the whole wave: e, end are uniform, lane group `sub` takes every (64 / LPR)-th entry and the
//          caller adds the groups
//   !WAVE  it belongs to the lane group: e, end may differ between the groups; all lanes of the wave take part
// U loads per lane are issued before the first is consumed, also at the end of a row (entries beyond it are masked out, not
// loaded): a row of 10 entries costs two round trips to memory and not one per entry, which bounds the launches of
// low-degree graphs.  Lanes beyond the row's last vector load the first one instead (the same line, never stored).
//   LIVE   rows of X that a.live does not name are zero and not read (see LIVE_BYTES below).  The bit of an entry is looked up one
//          chunk ahead and its index two, so that no trip waits for them.
__device__ __forceinline__ bool row_live(const SpmmArgs &a, int r) { return (a.live.bits[r >> 5] >> (r & 31)) & 1u; }

template <bool BF16, bool W, bool WAVE, int E, int LPR, int NV, int U, bool LIVE>
__device__ __forceinline__ void accumulate_row(const SpmmArgs &a, uint32_t e, uint32_t end, int lane, int elem0,
                                               float (&acc)[NV][E]) {
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int G = 64 / LPR;
    uint32_t off[NV];                               // the lane's place inside a feature row
#pragma unroll
    for (int v = 0; v < NV; ++v) off[v] = elem0 + v * LPR * E < a.F_lim ? static_cast<uint32_t>(elem0 + v * LPR * E) * ES : 0u;

    if constexpr (G == 1) {     // one entry per instruction: its row address is scalar
        for (; e < end; e += 64) {
            int n = static_cast<int>(end - e < 64u ? end - e : 64u);
            int c = 0, w = 0;
            bool on = false;
            if (lane < n) {
                c = a.idx[e + lane];
                if constexpr (W) w = __float_as_int(a.wt[e + lane]);
                if constexpr (LIVE) on = row_live(a, c);
            }
            if constexpr (LIVE) {       // the live entries first, in their order
                const uint64_t m = __ballot(on);
                const int before = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
                n = __popcll(m);
                const int to = 4 * (on ? before : n + lane - before);       // a permutation of the wave
                c = __builtin_amdgcn_ds_permute(to, c);
                if constexpr (W) w = __builtin_amdgcn_ds_permute(to, w);
            }
            int t = 0;
            for (; t + U <= n; t += U) {
                RawVec<BF16, E> x[U][NV];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const char *p = a.X + static_cast<int64_t>(__builtin_amdgcn_readlane(c, t + u)) * a.ldx_bytes;
#pragma unroll
                    for (int v = 0; v < NV; ++v) load_raw<BF16, E>(p + off[v], x[u][v]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float wu = 1.f;
                    if constexpr (W) wu = __int_as_float(__builtin_amdgcn_readlane(w, t + u));
#pragma unroll
                    for (int v = 0; v < NV; ++v) fma_raw<BF16, W, E>(wu, x[u][v], acc[v]);
                }
            }
            if (t < n) {        // the last U - 1 entries at most, in flight together as well
                RawVec<BF16, E> x[U - 1][NV];
#pragma unroll
                for (int u = 0; u < U - 1; ++u) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) zero_raw<BF16, E>(x[u][v]);
                    if (t + u < n) {
                        const char *p = a.X + static_cast<int64_t>(__builtin_amdgcn_readlane(c, t + u)) * a.ldx_bytes;
#pragma unroll
                        for (int v = 0; v < NV; ++v) load_raw<BF16, E>(p + off[v], x[u][v]);
                    }
                }
#pragma unroll
                for (int u = 0; u < U - 1; ++u) {
                    float wu = 1.f;
                    if constexpr (W) wu = __int_as_float(__builtin_amdgcn_readlane(w, (t + u) & 63));
#pragma unroll
                    for (int v = 0; v < NV; ++v) fma_raw<BF16, W, E>(wu, x[u][v], acc[v]);
                }
            }
        }
        return;
    }

    static_assert(G == 1 || NV == 1, "rows narrower than a wave are one vector per lane");
    constexpr int NQ = LPR < U ? U / LPR : 1;       // indices per lane and chunk
    constexpr int CH = LPR * NQ;                    // entries of a lane group per chunk
    constexpr uint32_t STEP = WAVE ? CH * G : CH;   // distance of a row's chunks
    const int sub = lane / LPR;
    const uint32_t mine = WAVE ? lane : lane % LPR, lanes = WAVE ? 64 : LPR;
    // entry k of the group: held by lane first + (k % LPR) * (WAVE ? G : 1), index register k / LPR
    const int first4 = 4 * (WAVE ? sub : sub * LPR);
    constexpr int STRIDE4 = 4 * (WAVE ? G : 1);
    const char *xbase = a.X + off[0];
    const uint32_t ld = static_cast<uint32_t>(a.ldx_bytes);
    int c[NQ], w[NQ];
    int cr[NQ];                     // LIVE: the next chunk's indices, not yet looked up
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const uint32_t i = e + q * lanes + mine;
        c[q] = i < end ? a.idx[i] : (LIVE ? -1 : 0);
        if constexpr (W) w[q] = i < end ? __float_as_int(a.wt[i]) : 0;
        if constexpr (LIVE) {
            cr[q] = i + STEP < end ? a.idx[i + STEP] : -1;
            if (c[q] >= 0 && !row_live(a, c[q])) c[q] = -1;
        }
    }
    while (WAVE ? e < end : __any(e < end)) {
        // entries the group still has (may exceed a chunk)
        const int n = e < end ? (WAVE ? (static_cast<int>(end - e) - sub + G - 1) / G : static_cast<int>(end - e)) : 0;
        e += STEP;
        int cn[NQ], wn[NQ];
        uint32_t ln[NQ];            // the word with the bit of cr
        auto trip = [&](int t, bool prefetch) __attribute__((always_inline)) {
            RawVec<BF16, E> x[U];
            int at = first4 + STRIDE4 * t;
            asm volatile("" : "+v"(at));    // formed here: the exchanges' constant distances stay immediate offsets
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t cj = __builtin_amdgcn_ds_bpermute(at + STRIDE4 * (u % LPR), c[NQ > 1 ? u / LPR : 0]);
                zero_raw<BF16, E>(x[u]);
                if (t + u < n && (!LIVE || static_cast<int>(cj) >= 0)) load_raw<BF16, E>(xbase + static_cast<uint64_t>(cj) * ld, x[u]);
            }
            if (prefetch) {             // the next chunk's indices: in flight behind the gathers, needed after them
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const uint32_t i = e + q * lanes + mine, i2 = LIVE ? i + STEP : i;
                    if constexpr (LIVE) ln[q] = cr[q] >= 0 ? a.live.bits[cr[q] >> 5] : 0u;
                    cn[q] = i2 < end ? a.idx[i2] : (LIVE ? -1 : 0);
                    if constexpr (W) wn[q] = i < end ? __float_as_int(a.wt[i]) : 0;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float wu = 1.f;
                if constexpr (W) wu = __int_as_float(__builtin_amdgcn_ds_bpermute(at + STRIDE4 * (u % LPR), w[NQ > 1 ? u / LPR : 0]));
                fma_raw<BF16, W, E>(wu, x[u], acc[0]);
            }
        };
        trip(0, true);
        if constexpr (CH > U) {
#pragma unroll 1
            for (int t = U; t < CH; t += U) {
                if (!__any(t < n)) break;
                trip(t, false);
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            if constexpr (LIVE) {
                c[q] = (ln[q] >> (cr[q] & 31)) & 1u ? cr[q] : -1;
                cr[q] = cn[q];
            } else {
                c[q] = cn[q];
            }
            if constexpr (W) w[q] = wn[q];
        }
    }
}

// adds the lane groups of a wave (a butterfly: the same order in every lane)
template <int E, int LPR, int NV>
__device__ __forceinline__ void add_lane_groups(float (&acc)[NV][E]) {
#pragma unroll
    for (int d = LPR; d < 64; d <<= 1)
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int j = 0; j < E; ++j) acc[v][j] += __shfl_xor(acc[v][j], d);
}

// Rows of the gathered matrix that are known to be zero (the loss gradient outside the training mask) are not read where the
// launch is bound by the fabric behind the L2s: rows of CROWDED_ROW entries and more on average, gathered from a matrix that the
// L2s do not keep.  980 k rows x 50 entries, 47 floats, 60 % of the rows live: 1630 -> 1133 us.  Not taken: 306 k rows x 13 entries
// (271 against 264 us), and the column-blocked kernel, which the L2s feed (60 k x 500 entries, 41 floats: 364 against 361).
// Above LIVE_SHARE of live rows the look-up costs more than the rows it saves (all of them live: 1920 us) and the launch reads
// every row.
constexpr int64_t LIVE_BYTES = int64_t(16) << 20;
constexpr float LIVE_SHARE = 0.85f;

// Scale, accumulate, bias, ReLU and store of E consecutive features of one output row.
template <bool OBF16, int E>
__device__ __forceinline__ void store_row(const SpmmArgs &a, int row, int f0, const float (&acc)[E]) {
    constexpr int ES = OBF16 ? 2 : 4;
    if (f0 >= a.F) return;
    char *yrow = a.Y + static_cast<int64_t>(row) * a.ldy_bytes;
    const float oscale = a.out_scale ? a.out_scale[row] : 1.f;
    const bool accumulate = row < a.acc_rows;
    const char *mrow = a.mask ? a.mask + static_cast<int64_t>(row) * a.ldm_bytes : nullptr;
    float y[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        float t = acc[j] * oscale;
        if (f0 + j < a.F) {
            if (accumulate) t += load_one<OBF16>(yrow + static_cast<int64_t>(f0 + j) * ES);
            if (a.bias) t += a.bias[f0 + j];
            if (mrow && !(load_one<OBF16>(mrow + static_cast<int64_t>(f0 + j) * ES) > 0.f)) t = 0.f;
        }
        if (a.relu) t = t > 0.f ? t : 0.f;
        y[j] = t;
    }
    if (f0 + E <= a.F) {
        store_elems<OBF16, E>(yrow + static_cast<int64_t>(f0) * ES, y);
    } else {
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (f0 + j < a.F) store_one<OBF16>(yrow + static_cast<int64_t>(f0 + j) * ES, y[j]);
    }
}

// What wave `w` of a launch works on: one of the first n_wave items, or 64 / LPR of the others, one per lane group.
template <bool BF16, bool OBF16, bool W, int E, int LPR, int NV, bool LIVE = false>
__device__ __forceinline__ void wave_items(const SpmmArgs &a, int64_t w, int lane) {
    constexpr int G = 64 / LPR;
    constexpr int U = (NV == 1) ? 8 : 4;
    constexpr int PASS = LPR * E * NV;
    const bool by_wave = G == 1 || w < a.n_wave;
    int64_t item = w;
    bool stores = true;
    if (!by_wave) {
        item = a.n_wave + (item - a.n_wave) * G + lane / LPR;
        stores = item < a.n_items;
    } else if constexpr (G > 1) {
        stores = lane < LPR;
    }
    RowItem it{0, 0u, 0u, 0u};
    if (by_wave || stores) it = a.items[item];

    for (int pass = 0; pass < a.F_lim; pass += PASS) {
        const int elem0 = pass + lane % LPR * E;
        float acc[NV][E];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int j = 0; j < E; ++j) acc[v][j] = 0.f;
        if (by_wave) {
            accumulate_row<BF16, W, true, E, LPR, NV, U, LIVE>(a, it.beg, it.beg + it.cnt, lane, elem0, acc);
            if constexpr (G > 1) add_lane_groups<E, LPR, NV>(acc);
        } else if constexpr (G > 1) {
            accumulate_row<BF16, W, false, E, LPR, NV, U, LIVE>(a, it.beg, it.beg + it.cnt, lane, elem0, acc);
        }
        if (!stores) continue;
        if (item < a.n_pieces) {
            float *prow = a.part + item * a.ldp;
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int f0 = elem0 + v * LPR * E;     // ldp covers whole vectors
                if (f0 < a.F) store_elems<false, E>(reinterpret_cast<char *>(prow + f0), acc[v]);
            }
        } else {
#pragma unroll
            for (int v = 0; v < NV; ++v) store_row<OBF16, E>(a, it.row, elem0 + v * LPR * E, acc[v]);
        }
    }
}

// Single-wave workgroups: a wave that shares a workgroup with a longer row would hold its slot until that one ends.  The
// launches are bound by how many gathers the resident waves keep in flight, then by the fabric behind the L2s: at least
// five (bf16) or six waves per SIMD are asked for (the bf16-in / fp32-out variants otherwise settle at four; six would spill
// in the bf16 variants: 7.46 against 7.06 ms for two launches of 980 k rows x 50 entries x 256 features).  W: entries have
// weights (a.wt), else every weight is 1.
template <bool BF16, bool OBF16, bool W, int E, int LPR, int NV, bool LIVE = false>
__global__ __launch_bounds__(64, NV < 3 ? (BF16 && LPR < 64 ? 5 : 6) : 1) void spmm_kernel(SpmmArgs a) {
    if (LIVE && a.live.count[0] <= LIVE_SHARE * static_cast<float>(a.n_in)) wave_items<BF16, OBF16, W, E, LPR, NV, LIVE>(a, blockIdx.x, threadIdx.x);
    else wave_items<BF16, OBF16, W, E, LPR, NV>(a, blockIdx.x, threadIdx.x);
}

// Workgroups [0, n_cut): one long row each, its entries shared by the waves and the partial sums added through LDS in wave
// order.  The rest: the short items, one wave after the other.  Serves small graphs, whose launch is over before the pieces
// of cut rows and the kernel that adds them would be, and the long rows where the caller brought no scratch for pieces.
template <int NV> constexpr int ROW_WAVES = NV == 1 ? 16 : 4;
template <bool BF16, bool OBF16, bool W, int E, int LPR, int NV>
__global__ __launch_bounds__(64 * ROW_WAVES<NV>) void spmm_rows_kernel(SpmmArgs a, const RowItem *cut, int n_cut, const RowItem *whole,
                                                                          int n_rows, int64_t n_waves) {
    constexpr int U = (NV == 1) ? 8 : 4;
    constexpr int PASS = LPR * E * NV;
    constexpr int NW = ROW_WAVES<NV>;
    __shared__ float red[NW - 1][NV * E][LPR];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (static_cast<int>(blockIdx.x) >= n_rows) {
        const int64_t w = static_cast<int64_t>(blockIdx.x - n_rows) * NW + wave;
        if (w < n_waves) wave_items<BF16, OBF16, W, E, LPR, NV>(a, w, lane);
        return;
    }
    const RowItem it = static_cast<int>(blockIdx.x) < n_cut ? cut[blockIdx.x] : whole[blockIdx.x - n_cut];
    const uint32_t end = it.beg + it.cnt, per = (it.cnt + NW - 1) / NW;
    const uint32_t e0 = wave * per < it.cnt ? it.beg + wave * per : end, e1 = end - e0 < per ? end : e0 + per;
    for (int pass = 0; pass < a.F_lim; pass += PASS) {
        const int elem0 = pass + lane % LPR * E;
        float acc[NV][E];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int j = 0; j < E; ++j) acc[v][j] = 0.f;
        accumulate_row<BF16, W, true, E, LPR, NV, U, false>(a, e0, e1, lane, elem0, acc);
        if constexpr (LPR < 64) add_lane_groups<E, LPR, NV>(acc);
        if (pass > 0) __syncthreads();
        if (wave > 0 && lane < LPR) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int j = 0; j < E; ++j) red[wave - 1][v * E + j][lane] = acc[v][j];
        }
        __syncthreads();
        if (wave == 0 && lane < LPR) {
#pragma unroll 3
            for (int p = 0; p < NW - 1; ++p)
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int j = 0; j < E; ++j) acc[v][j] += red[p][v * E + j][lane];
#pragma unroll
            for (int v = 0; v < NV; ++v) store_row<OBF16, E>(a, it.row, elem0 + v * LPR * E, acc[v]);
        }
    }
}

// ---------------------------------------------------------------------------------------------------
// Column-blocked variant for dense-degree operators whose gathered matrix is larger than an L2.
//
// A task is (source block cb, output position p, feature slice s): it sums the entries of row order[p] whose
// source lies in block cb, over one SLICE_BYTES-wide slice of the feature row, and stores the partial row to
// scratch.  The grid is laid out so that the workgroups running on one L2 domain at any moment share (cb, s):
// their gathers then address CB_ROWS * SLICE_BYTES = 4 MB, the size of that L2.  Workgroup b runs on domain
// b % NUM_XCD; the slices (times H interleaved shares of the rows when there are fewer slices than domains)
// are dealt to the domains, and each domain sweeps its units block by block.  Within a (unit, block) phase the
// positions come heaviest first in three classes: a whole workgroup per task, a wave per task, and eight
// tasks per wave (one per 8-lane group).  A second kernel sums the partials of a row over the blocks in a
// fixed order and applies the epilogue.
struct SpmmBlockedArgs {
    const uint32_t *off;         // [ncb*n_out + 1]
    const int2 *ew;              // [nnz] {source row, weight bits}
    const uint16_t *src;         // [nnz] source row inside its block: read instead of ew (every weight taken as 1) when not null
    int64_t n_out, n_long, n_mid;
    int ncb, H;                  // source blocks, row shares per slice
    int64_t RG_long, RG_mid, RG; // workgroups per (unit, block): long class, medium class, all
    const char *X;
    uint32_t ld16;               // row pitch of X in 16-byte units
    int F_lim;
    float *part;                 // [ncb*n_out][ldp] partial rows
    int64_t ldp;
};

// entry i of block cb: {source row, weight bits}; from the 2-byte list when the weights are not needed (uniform over
// the launch)
__device__ __forceinline__ int2 blocked_entry(const SpmmBlockedArgs &b, int cb, uint32_t i) {
    return b.src ? make_int2(cb * CB_ROWS + b.src[i], 0x3f800000) : b.ew[i];
}

constexpr int B_LPR = SLICE_BYTES / 16;      // lanes that cover one slice with 16-byte loads
constexpr int B_GROUPS = 64 / B_LPR;         // entries (or rows) a wave works on at the same time
constexpr int B_MID_PER_WAVE = 4;            // consecutive medium positions one wave handles
constexpr int B_SHORT_PER_GROUP = 2;         // consecutive short positions one lane group handles
// entries per trip of a lane group when the entries carry no weights (bf16 rows widen to twice the registers)
template <bool BF16> constexpr int B_SHORT_DEPTH = BF16 ? 8 : 16;
constexpr int B_MID_PER_WG = 4 * B_MID_PER_WAVE;
constexpr int B_SHORT_PER_WG = 4 * B_GROUPS * B_SHORT_PER_GROUP;
static_assert(B_LPR == 8, "lane-group shuffles below assume 8-lane groups");

// value of `v` in lane k of the caller's 8-lane group (ds_swizzle, bit-mask mode: lane = (lane & 0x18) | k)
__device__ __forceinline__ int group_bcast(int v, int k) {
    switch (k) {
        case 0: return __builtin_amdgcn_ds_swizzle(v, 0x0018);
        case 1: return __builtin_amdgcn_ds_swizzle(v, 0x0038);
        case 2: return __builtin_amdgcn_ds_swizzle(v, 0x0058);
        case 3: return __builtin_amdgcn_ds_swizzle(v, 0x0078);
        case 4: return __builtin_amdgcn_ds_swizzle(v, 0x0098);
        case 5: return __builtin_amdgcn_ds_swizzle(v, 0x00b8);
        case 6: return __builtin_amdgcn_ds_swizzle(v, 0x00d8);
        default: return __builtin_amdgcn_ds_swizzle(v, 0x00f8);
    }
}

// All 64 lanes work on ONE row: entries [e0, e1) are read 64 at a time (coalesced), lane group g then takes
// entries g, g+8, ... of the chunk, so up to eight 16-byte-per-lane feature loads are in flight per wave.
// On return every lane of group g holds the sum over that group's entries; the caller adds the groups.
template <bool BF16, bool WEIGHTED, int E>
__device__ __forceinline__ void blocked_row_accumulate(const SpmmBlockedArgs &b, int cb, uint32_t e0, uint32_t e1, int lane,
                                                       const char *xbase, bool ok, float (&acc)[E]) {
    const int grp = lane / B_LPR;
    if constexpr (!WEIGHTED) {
        // bare row numbers: NC chunks of 64 entries per trip (NC * 8 feature loads in flight per lane), plain sums
        // (NC = 2 costs a wave per SIMD in registers and 2 % of the launch: measured)
        constexpr int NC = 1;
        const int rowbase = cb * CB_ROWS;
        int cur[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) cur[q] = (e0 + 64 * q + lane < e1) ? rowbase + b.src[e0 + 64 * q + lane] : 0;
        for (uint32_t c0 = e0; c0 < e1; c0 += 64 * NC) {
            int coff[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) coff[q] = static_cast<int>(__umul24(static_cast<uint32_t>(cur[q]), b.ld16));
#pragma unroll
            for (int q = 0; q < NC; ++q)
                cur[q] = (c0 + 64 * (NC + q) + lane < e1) ? rowbase + b.src[c0 + 64 * (NC + q) + lane] : 0;
            const int cnt = static_cast<int>(e1 - c0 < 64u * NC ? e1 - c0 : 64u * NC);
            float xk[NC * B_GROUPS][E];
#pragma unroll
            for (int k = 0; k < NC * B_GROUPS; ++k) {
                const int src = (k % B_GROUPS) * B_GROUPS + grp;             // lane that holds the entry, in chunk k / B_GROUPS
                const uint32_t ck = static_cast<uint32_t>(__shfl(coff[k / B_GROUPS], src));
                if ((k / B_GROUPS) * 64 + src < cnt && ok) {
                    load_elems<BF16, E>(xbase + (static_cast<uint64_t>(ck) << 4), xk[k]);
                } else {
#pragma unroll
                    for (int j = 0; j < E; ++j) xk[k][j] = 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < NC * B_GROUPS; ++k)
#pragma unroll
                for (int j = 0; j < E; ++j) acc[j] += xk[k][j];
        }
        return;
    }
    int2 pr = make_int2(0, 0);
    if (e0 + lane < e1) pr = blocked_entry(b, cb, e0 + lane);
    for (uint32_t c0 = e0; c0 < e1; c0 += 64) {
        const int coff = static_cast<int>(__umul24(static_cast<uint32_t>(pr.x), b.ld16));   // 16-byte units
        const int wbits = pr.y;                                                               // 0 beyond the end
        pr = make_int2(0, 0);
        if (c0 + 64 + lane < e1) pr = blocked_entry(b, cb, c0 + 64 + lane);      // next chunk's entries are on their way early
        const int cnt = static_cast<int>(e1 - c0 < 64u ? e1 - c0 : 64u);
        float xk[B_GROUPS][E], wk[B_GROUPS];
#pragma unroll
        for (int k = 0; k < B_GROUPS; ++k) {
            if (k * B_GROUPS < cnt) {      // wave-uniform
                const int src = k * B_GROUPS + grp;
                const uint32_t ck = static_cast<uint32_t>(__shfl(coff, src));
                wk[k] = __int_as_float(__shfl(wbits, src));
                if (src < cnt && ok) {
                    load_elems<BF16, E>(xbase + (static_cast<uint64_t>(ck) << 4), xk[k]);
                } else {
#pragma unroll
                    for (int j = 0; j < E; ++j) xk[k][j] = 0.f;
                }
            }
        }
#pragma unroll
        for (int k = 0; k < B_GROUPS; ++k)
            if (k * B_GROUPS < cnt) {
#pragma unroll
                for (int j = 0; j < E; ++j) acc[j] = fmaf(wk[k], xk[k][j], acc[j]);
            }
    }
}

template <int E>
__device__ __forceinline__ void add_groups(float (&acc)[E]) {
#pragma unroll
    for (int off = B_LPR; off < 64; off <<= 1)
#pragma unroll
        for (int j = 0; j < E; ++j) acc[j] += __shfl_xor(acc[j], off);
}

// WEIGHTED: entries come with their weights (b.ew); otherwise as bare block-local row numbers (b.src), every weight 1.
template <bool BF16, bool WEIGHTED>
__global__ __launch_bounds__(256) void spmm_blocked_kernel(SpmmBlockedArgs b) {
    constexpr int E = BF16 ? 8 : 4;
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int SLICE = B_LPR * E;
    __shared__ float red[3][E][B_LPR];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int l = lane % B_LPR, grp = lane / B_LPR;
    const int x = blockIdx.x % NUM_XCD;
    int64_t q = blockIdx.x / NUM_XCD;
    int64_t r = q % b.RG;
    q /= b.RG;
    const int cb = static_cast<int>(q % b.ncb);
    const int64_t u = x + NUM_XCD * (q / b.ncb);     // unit = (slice, share)
    const int s = static_cast<int>(u / b.H), h = static_cast<int>(u % b.H);
    const int elem0 = s * SLICE + l * E;
    const bool ok = elem0 < b.F_lim;
    const char *xbase = b.X + static_cast<int64_t>(elem0) * ES;
    const int64_t tbase = static_cast<int64_t>(cb) * b.n_out;

    if (r < b.RG_long) {
        // ---- a whole workgroup on one task: the four waves take quarters of the group, summed through LDS
        const int64_t p = r * b.H + h;
        if (p >= b.n_long) return;                   // uniform over the workgroup
        const uint32_t e0 = b.off[tbase + p], e1 = b.off[tbase + p + 1];
        if (e0 == e1) return;
        const uint32_t per = ((e1 - e0 + 3) / 4 + 63) / 64 * 64;
        uint32_t w0 = e0 + wave * per, w1 = w0 + per;
        if (w0 > e1) w0 = e1;
        if (w1 > e1) w1 = e1;
        float acc[E];
#pragma unroll
        for (int j = 0; j < E; ++j) acc[j] = 0.f;
        blocked_row_accumulate<BF16, WEIGHTED, E>(b, cb, w0, w1, lane, xbase, ok, acc);
        add_groups<E>(acc);
        if (wave > 0 && lane < B_LPR) {
#pragma unroll
            for (int j = 0; j < E; ++j) red[wave - 1][j][lane] = acc[j];
        }
        __syncthreads();
        if (wave == 0 && lane < B_LPR) {
#pragma unroll
            for (int wv = 0; wv < 3; ++wv)
#pragma unroll
                for (int j = 0; j < E; ++j) acc[j] += red[wv][j][lane];
            store_elems<false, E>(reinterpret_cast<char *>(b.part + (tbase + p) * b.ldp + elem0), acc);
        }
        return;
    }
    r -= b.RG_long;
    if (r < b.RG_mid) {
        // ---- one wave per task
        const int64_t p0 = b.n_long + (r * b.H + h) * B_MID_PER_WG + wave * B_MID_PER_WAVE;
        for (int i = 0; i < B_MID_PER_WAVE; ++i) {
            const int64_t p = p0 + i;
            if (p >= b.n_mid) break;
            const uint32_t e0 = b.off[tbase + p], e1 = b.off[tbase + p + 1];
            if (e0 == e1) continue;
            float acc[E];
#pragma unroll
            for (int j = 0; j < E; ++j) acc[j] = 0.f;
            blocked_row_accumulate<BF16, WEIGHTED, E>(b, cb, e0, e1, lane, xbase, ok, acc);
            add_groups<E>(acc);
            if (lane < B_LPR) store_elems<false, E>(reinterpret_cast<char *>(b.part + (tbase + p) * b.ldp + elem0), acc);
        }
        return;
    }
    r -= b.RG_mid;
    // ---- eight tasks per wave: each 8-lane group owns one position and walks its entries 8 per trip (one index
    // load per group, then 8 independent feature loads in flight)
    const int64_t p0 = b.n_mid + (r * b.H + h) * B_SHORT_PER_WG + wave * (B_GROUPS * B_SHORT_PER_GROUP);
    for (int i = 0; i < B_SHORT_PER_GROUP; ++i) {
        const int64_t p = p0 + i * B_GROUPS + grp;
        uint32_t e = 0, e1 = 0;
        if (p < b.n_out) { e = b.off[tbase + p]; e1 = b.off[tbase + p + 1]; }
        const bool any_entry = e < e1;
        float acc[E];
#pragma unroll
        for (int j = 0; j < E; ++j) acc[j] = 0.f;
        if constexpr (!WEIGHTED) {
            // bare row numbers, B_SHORT_DEPTH entries per trip: each lane fetches an eighth of them, the group exchanges
            // them and every lane has that many feature loads in flight; the sums need no multiply
            constexpr int NQ = B_SHORT_DEPTH<BF16> / B_LPR;
            const int rowbase = cb * CB_ROWS;
            int cur[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) cur[q] = (e + q * B_LPR + l < e1) ? rowbase + b.src[e + q * B_LPR + l] : 0;
            while (__any(e < e1)) {
                const int n = e < e1 ? static_cast<int>(e1 - e) : 0;    // entries this group still has (may exceed a trip)
                int coff[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) coff[q] = static_cast<int>(__umul24(static_cast<uint32_t>(cur[q]), b.ld16));
                e += B_SHORT_DEPTH<BF16>;
#pragma unroll
                for (int q = 0; q < NQ; ++q) cur[q] = (e + q * B_LPR + l < e1) ? rowbase + b.src[e + q * B_LPR + l] : 0;
                float xk[B_SHORT_DEPTH<BF16>][E];
#pragma unroll
                for (int k = 0; k < B_SHORT_DEPTH<BF16>; ++k) {
                    const uint32_t ck = static_cast<uint32_t>(group_bcast(coff[k / B_LPR], k % B_LPR));
                    if (k < n && ok) {
                        load_elems<BF16, E>(xbase + (static_cast<uint64_t>(ck) << 4), xk[k]);
                    } else {
#pragma unroll
                        for (int j = 0; j < E; ++j) xk[k][j] = 0.f;
                    }
                }
#pragma unroll
                for (int k = 0; k < B_SHORT_DEPTH<BF16>; ++k)
#pragma unroll
                    for (int j = 0; j < E; ++j) acc[j] += xk[k][j];
            }
            if (any_entry) store_elems<false, E>(reinterpret_cast<char *>(b.part + (tbase + p) * b.ldp + elem0), acc);
            continue;
        }
        int2 pr = make_int2(0, 0);
        if (e + l < e1) pr = blocked_entry(b, cb, e + l);
        while (__any(e < e1)) {
            const int coff = static_cast<int>(__umul24(static_cast<uint32_t>(pr.x), b.ld16));   // in 16-byte units
            const int wbits = pr.y;
            const int n = e < e1 ? static_cast<int>(e1 - e) : 0;    // entries this group still has (may exceed 8)
            e += B_LPR;
            pr = make_int2(0, 0);
            if (e + l < e1) pr = blocked_entry(b, cb, e + l);                       // next trip's entries are on their way early
            float xk[B_LPR][E], wk[B_LPR];
#pragma unroll
            for (int k = 0; k < B_LPR; ++k) {
                const uint32_t ck = static_cast<uint32_t>(group_bcast(coff, k));
                wk[k] = __int_as_float(group_bcast(wbits, k));
                if (k < n && ok) {
                    load_elems<BF16, E>(xbase + (static_cast<uint64_t>(ck) << 4), xk[k]);
                } else {
#pragma unroll
                    for (int j = 0; j < E; ++j) xk[k][j] = 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < B_LPR; ++k)
#pragma unroll
                for (int j = 0; j < E; ++j) acc[j] = fmaf(wk[k], xk[k][j], acc[j]);
        }
        if (any_entry) store_elems<false, E>(reinterpret_cast<char *>(b.part + (tbase + p) * b.ldp + elem0), acc);
    }
}

struct SpmmReduceArgs {
    const uint32_t *off;
    const int32_t *order;
    const float *out_scale;
    const float *part;
    int64_t ldp, n_out;
    int ncb;
    char *Y;
    int64_t ldy_bytes;
    int F;
    const float *bias;
    int relu, acc_rows;
    const char *mask;
    int64_t ldm_bytes;
};

// one thread per (position, four consecutive features)
template <bool OBF16>
__global__ __launch_bounds__(256) void spmm_blocked_reduce_kernel(SpmmReduceArgs a) {
    constexpr int ES = OBF16 ? 2 : 4;
    const int chunks = (a.F + 3) / 4;
    const int64_t tid = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t p = tid / chunks;
    if (p >= a.n_out) return;
    const int f0 = static_cast<int>(tid % chunks) * 4;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int cb = 0; cb < a.ncb; ++cb) {
        const int64_t t = static_cast<int64_t>(cb) * a.n_out + p;
        if (a.off[t + 1] == a.off[t]) continue;      // empty group: its partial row was never written
        const float4 v = *reinterpret_cast<const float4 *>(a.part + t * a.ldp + f0);
        acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    const int row = a.order[p];
    const float oscale = a.out_scale ? a.out_scale[row] : 1.f;
    char *yrow = a.Y + static_cast<int64_t>(row) * a.ldy_bytes;
    float y[4] = {acc.x * oscale, acc.y * oscale, acc.z * oscale, acc.w * oscale};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (f0 + j < a.F) {
            if (row < a.acc_rows) y[j] += load_one<OBF16>(yrow + static_cast<int64_t>(f0 + j) * ES);
            if (a.bias) y[j] += a.bias[f0 + j];
            if (a.mask && !(load_one<OBF16>(a.mask + row * a.ldm_bytes + static_cast<int64_t>(f0 + j) * ES) > 0.f)) y[j] = 0.f;
        }
        if (a.relu) y[j] = y[j] > 0.f ? y[j] : 0.f;
    }
    if (f0 + 4 <= a.F) {
        if constexpr (OBF16) {
            uint2 v;
            v.x = f32_to_bf16_bits(y[0]) | (f32_to_bf16_bits(y[1]) << 16);
            v.y = f32_to_bf16_bits(y[2]) | (f32_to_bf16_bits(y[3]) << 16);
            *reinterpret_cast<uint2 *>(yrow + static_cast<int64_t>(f0) * ES) = v;
        } else {
            *reinterpret_cast<float4 *>(yrow + static_cast<int64_t>(f0) * ES) = make_float4(y[0], y[1], y[2], y[3]);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (f0 + j < a.F) store_one<OBF16>(yrow + static_cast<int64_t>(f0 + j) * ES, y[j]);
    }
}

// Geometry of the blocked launch for a width-F operand; ok == false when the blocked kernel does not apply.
struct BlockedGeom {
    bool ok = false;
    int ns = 0, H = 0;
    int64_t U = 0, RG_long = 0, RG_mid = 0, RG = 0, ldp = 0, grid = 0;
    size_t ws = 0;
};

static BlockedGeom blocked_geom(const SpOp &op, int F, int dtype) {
    BlockedGeom g;
    if (op.ncb == 0 || F <= 0) return g;
    const int slice = SLICE_BYTES / elem_bytes(dtype);
    if (F < slice) return g;                         // narrow rows: the whole operand is small, one pass does
    if (op.n_in >= (int64_t(1) << 24)) return g;     // the kernel forms source offsets with 24-bit multiplies
    g.ns = (F + slice - 1) / slice;
    int gcd = g.ns, t = NUM_XCD;
    while (t) { const int m = gcd % t; gcd = t; t = m; }
    g.H = NUM_XCD / gcd;
    g.U = static_cast<int64_t>(g.ns) * g.H / NUM_XCD;
    auto per_share = [&](int64_t positions, int per_wg) { return ((positions + per_wg - 1) / per_wg + g.H - 1) / g.H; };
    g.RG_long = per_share(op.b_long, 1);
    g.RG_mid = per_share(op.b_mid - op.b_long, B_MID_PER_WG);
    g.RG = g.RG_long + g.RG_mid + per_share(op.n_out - op.b_mid, B_SHORT_PER_WG);
    g.ldp = static_cast<int64_t>(g.ns) * slice;
    g.grid = NUM_XCD * g.U * op.ncb * g.RG;
    if (g.grid <= 0 || g.grid >= (int64_t(1) << 31)) return g;
    g.ws = align_up(static_cast<size_t>(op.ncb) * op.n_out * g.ldp * sizeof(float), 256);
    g.ok = true;
    return g;
}

static int64_t pieces_ldp(int F) { return (static_cast<int64_t>(F) + 7) / 8 * 8; }

size_t spmm_ws_bytes(const SpOp &op, int F, int dtype) {
    const BlockedGeom g = blocked_geom(op, F, dtype);
    const int64_t pieces = std::max(op.list.n_pieces, op.list_sub.n_pieces);
    const size_t cut = F > 0 ? static_cast<size_t>(pieces) * pieces_ldp(F) * sizeof(float) : 0;
    return std::max<size_t>(g.ok ? g.ws : 0, cut);
}

template <bool BF16, bool OBF16>
static int launch_blocked(const SpOp &op, const BlockedGeom &g, const SpmmArgs &a, float *part, hipStream_t st) {
    SpmmBlockedArgs b;
    b.off = op.b_off; b.ew = op.b_ew; b.src = (a.wt == nullptr) ? op.b_src : nullptr; b.n_out = op.n_out; b.n_long = op.b_long; b.n_mid = op.b_mid;
    b.ncb = op.ncb; b.H = g.H; b.RG_long = g.RG_long; b.RG_mid = g.RG_mid; b.RG = g.RG;
    b.X = a.X; b.ld16 = static_cast<uint32_t>(a.ldx_bytes >> 4); b.F_lim = a.F_lim;
    b.part = part; b.ldp = g.ldp;
    if (b.src) hipLaunchKernelGGL((spmm_blocked_kernel<BF16, false>), dim3(static_cast<unsigned>(g.grid)), dim3(256), 0, st, b);
    else hipLaunchKernelGGL((spmm_blocked_kernel<BF16, true>), dim3(static_cast<unsigned>(g.grid)), dim3(256), 0, st, b);
    CG_HIP(hipGetLastError());
    SpmmReduceArgs r;
    r.off = op.b_off; r.order = op.order; r.out_scale = op.out_scale; r.part = part; r.ldp = g.ldp; r.n_out = op.n_out;
    r.ncb = op.ncb; r.Y = a.Y; r.ldy_bytes = a.ldy_bytes; r.F = a.F; r.bias = a.bias; r.relu = a.relu;
    r.acc_rows = a.acc_rows; r.mask = a.mask; r.ldm_bytes = a.ldm_bytes;
    const int64_t threads = op.n_out * ((a.F + 3) / 4);
    hipLaunchKernelGGL((spmm_blocked_reduce_kernel<OBF16>), dim3(static_cast<unsigned>((threads + 255) / 256)), dim3(256),
                       0, st, r);
    CG_HIP(hipGetLastError());
    return CAPGNN_OK;
}

// Completes the cut rows: sums the pieces of a row in a fixed order (blockDim.y strided groups, then the groups in order)
// and applies the same epilogue as spmm_kernel.  One workgroup per (row, 64 features).
template <bool OBF16>
__global__ void spmm_pieces_finish_kernel(SpmmArgs a, const RowItem *cut, const int32_t *piece_first) {
    __shared__ float red[16][64];
    const int k = blockIdx.x, f = blockIdx.y * 64 + threadIdx.x;
    const int row = cut[k].row, q1 = piece_first[k + 1], step = blockDim.y;
    float s = 0.f;
    if (f < a.F) {
        int q = piece_first[k] + threadIdx.y;
        for (; q + 7 * step < q1; q += 8 * step) {         // eight loads in flight
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = a.part[static_cast<int64_t>(q + u * step) * a.ldp + f];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; q < q1; q += step) s += a.part[static_cast<int64_t>(q) * a.ldp + f];
    }
    red[threadIdx.y][threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.y != 0 || f >= a.F) return;
    float acc[1] = {0.f};
    for (int y = 0; y < step; ++y) acc[0] += red[y][threadIdx.x];
    store_row<OBF16, 1>(a, row, f, acc);
}

// How long a row may be that one lane group walks alone.  A group takes about a microsecond for eight entries, so a row of T
// entries ends T / 8 us after it began: T follows the time the launch needs anyway (its gathers at 5 TB/s), from 16 (a
// 40 k-entry launch of 8 features: 4.4 us with 16, 8.0 with 64, 12 with 128) to 128 (6 M entries of 47 bf16 features: 150 us
// with 16, 110 with 64, 106 with 128).
static int group_row_entries(int64_t nnz, int64_t row_bytes) {
    const double us = static_cast<double>(nnz) * row_bytes / 5e6;
    int t = 16;
    while (t < 128 && t < us) t *= 2;
    return t;
}

// Unused LDS asked for by the launches whose rows average at least CROWDED_ROW entries of at least CROWDED_BYTES: twelve
// waves per compute unit instead of 20 to 28.  Twelve keep the fabric behind the L2s busy with such rows, and fewer rows
// under way at a time leave more of the L2s to the hubs: 980 k rows x 50 entries, 256 bf16 features 3.61 -> 3.46 ms, 128
// features 1.81 -> 1.70, 64 float features 1.88 -> 1.79; 400 k rows x 35 entries 2 to 3 %, 200 k rows x 100 entries 4 to 10 %.
// Shorter rows need the waves to hide their start and end (13 entries x 256 float features: 0.60 -> 0.63 ms), narrower ones to
// keep enough requests in flight (47 bf16 features: 0.10 -> 0.115).  It costs where most gathers hit the L2s anyway: Zipf halo
// columns, 300 k rows x 50 entries x 256 bf16 features 0.73 -> 0.755 ms, 1 M rows x 40 entries x 512 4.66 -> 4.86.
constexpr int CROWDED_ROW = 32, CROWDED_BYTES = 192, CROWDED_LDS = 13312;

// Graphs of at most ROWS_NNZ entries with rows to cut run as one launch of spmm_rows_kernel: the second launch costs more than
// what the finer cut saves (the three aggregations of a 10 k-vertex GraphSAGE epoch 37 -> 31 us, of a 22 k-vertex GIN epoch
// 65 -> 61, besides three launch gaps of 1-2 us).  That holds while the longest row, which one workgroup walks, ends with the
// launch.  A compute unit that has other rows as well gathers 50 GB/s for it (four waves, rows of several vectors per lane: 30);
// the rest of the launch takes its bytes at about 8.5 TB/s (short rows, cached) and the pieces' two launches about 5 us more.
// us as one launch and as pieces, 200 k entries x 41 floats: longest row of 1024 entries 8.2 / 9.5, 2048 9.1 / 8.7, 4096 14.6 /
// 9.1, 65536 182 / 13; x 256 floats: 1024 28 / 33, 2048 37 / 32, 16384 180 / 33; 900 k entries x 256: 4096 130 / 139, 8192 164 /
// 140, 200 k 2076 / 144.
constexpr int64_t ROWS_NNZ = int64_t(1) << 20;
static bool rows_in_one_launch(int64_t nnz, int64_t longest, int64_t row_bytes, int row_waves) {
    const double row_us = static_cast<double>(longest) * row_bytes / (row_waves >= 16 ? 5e4 : 3e4);
    return nnz <= ROWS_NNZ && row_us <= 5.0 + static_cast<double>(nnz) * row_bytes / 8.5e6;
}

// Rows below the cut that a launch of spmm_rows_kernel gives a workgroup each as well: a wave takes about a microsecond for a
// trip (its gathers under way at once), so those of at least two trips and of a quarter of what the launch's bytes need at 8.5 TB/s,
// while they and the cut rows are no more than the compute units.  us: 40 k entries x 128 floats 12.3 -> 7.3, the epoch of two
// layers around it 63.6 -> 59.3; an epoch of 420 k entries (50 and 128 floats) 202 -> 195; forward and backward of 77 k entries
// x 80 floats 22.3 -> 20.9.  With half of that time as the second bound the 420 k entries gain nothing, without one an epoch of
// 200 k entries x 128 floats goes 286 -> 288.  Trips of a wave matter: 32 bf16 features take 128 entries per trip, and rows of 32
// entries in workgroups of their own cost an epoch of 100 k such entries 109 -> 129.  Graphs without cut rows keep single-wave
// workgroups (490 k entries of 98 k short rows: an epoch 304 -> 332 in workgroups of sixteen).
static int64_t middling_rows(const ItemList &list, int64_t nnz, int64_t row_bytes, int trip) {
    const double trips = std::max(2.0, 0.25 * static_cast<double>(nnz) * row_bytes / 8.5e6);
    int64_t rows = 0;
    for (int t = 1024; t >= 32 && t >= trips * trip; t /= 2) {
        const int64_t m = list.first_below(t) - list.n_pieces;
        if (list.n_cut + m > NUM_CU) break;
        rows = m;
    }
    return rows;
}

// pieces: the caller brought scratch for the pieces of the cut rows
template <bool BF16, bool OBF16, bool W, int E, int LPR, int NV>
static int launch_cfg(SpmmArgs a, const ItemList &list, bool pieces, int64_t nnz, hipStream_t st) {
    constexpr int G = 64 / LPR, NW = ROW_WAVES<NV>;
    a.items = list.items; a.n_items = list.n_items; a.n_pieces = list.n_pieces;
    const int64_t row_bytes = static_cast<int64_t>(a.F_lim) * (BF16 ? 2 : 4);
    a.n_wave = G == 1 ? list.n_items : list.first_below(group_row_entries(nnz, row_bytes));
    const bool long_rows = nnz >= CROWDED_ROW * list.n_items && row_bytes >= CROWDED_BYTES;
    const bool one_launch = list.n_cut > 0 && (pieces ? rows_in_one_launch(nnz, list.longest, row_bytes, NW) : nnz <= ROWS_NNZ);
    pieces = pieces && !one_launch;
    const int64_t middling = one_launch ? middling_rows(list, nnz, row_bytes, G * (NV == 1 ? 8 : 4)) : 0;
    const RowItem *const whole = list.items + list.n_pieces;
    const int64_t rows = pieces ? 0 : list.n_cut + middling;        // given a workgroup each
    if (!pieces) {
        const int64_t skip = list.n_pieces + middling;
        a.items += skip; a.n_items -= skip; a.n_wave = std::max<int64_t>(a.n_wave - skip, 0); a.n_pieces = 0;
    }
    const int64_t waves = a.n_wave + (a.n_items - a.n_wave + G - 1) / G;
    if (rows > 0)
        hipLaunchKernelGGL((spmm_rows_kernel<BF16, OBF16, W, E, LPR, NV>),
                           dim3(static_cast<unsigned>(rows + (one_launch ? (waves + NW - 1) / NW : 0))), dim3(64 * NW), 0, st, a,
                           list.cut, static_cast<int>(list.n_cut), whole, static_cast<int>(rows), waves);
    if (!one_launch && waves > 0) {
        bool done = false;
        if constexpr (!BF16 && E > 1 && LPR > 4) {
            if (a.live.bits) {
                hipLaunchKernelGGL((spmm_kernel<BF16, OBF16, W, E, LPR, NV, true>), dim3(static_cast<unsigned>(waves)), dim3(64), 0, st, a);
                done = true;
            }
        }
        if (!done)
            hipLaunchKernelGGL((spmm_kernel<BF16, OBF16, W, E, LPR, NV>), dim3(static_cast<unsigned>(waves)), dim3(64),
                               long_rows ? CROWDED_LDS : 0, st, a);
    }
    if (pieces)
        hipLaunchKernelGGL((spmm_pieces_finish_kernel<OBF16>), dim3(static_cast<unsigned>(list.n_cut), (a.F + 63) / 64),
                           dim3(64, list.max_pieces > 64 ? 16 : 4), 0, st, a, list.cut, list.piece_first);
    CG_HIP(hipGetLastError());
    return CAPGNN_OK;
}

template <bool BF16, bool OBF16, bool W>
static int dispatch_w(const SpmmArgs &a, bool vec, const ItemList &list, bool pieces, int64_t nnz, hipStream_t st) {
    constexpr int EV = BF16 ? 8 : 4;
    if (vec) {
        const int nvec = a.F_lim / EV;
        if (nvec <= 4) return launch_cfg<BF16, OBF16, W, EV, 4, 1>(a, list, pieces, nnz, st);
        if (nvec <= 8) return launch_cfg<BF16, OBF16, W, EV, 8, 1>(a, list, pieces, nnz, st);
        if (nvec <= 16) return launch_cfg<BF16, OBF16, W, EV, 16, 1>(a, list, pieces, nnz, st);
        if (nvec <= 32) return launch_cfg<BF16, OBF16, W, EV, 32, 1>(a, list, pieces, nnz, st);
        if (nvec <= 64) return launch_cfg<BF16, OBF16, W, EV, 64, 1>(a, list, pieces, nnz, st);
        if (nvec <= 128) return launch_cfg<BF16, OBF16, W, EV, 64, 2>(a, list, pieces, nnz, st);
        return launch_cfg<BF16, OBF16, W, EV, 64, 3>(a, list, pieces, nnz, st);   // wider rows take several passes
    }
    if (a.F <= 64) return launch_cfg<BF16, OBF16, W, 1, 64, 1>(a, list, pieces, nnz, st);
    if (a.F <= 128) return launch_cfg<BF16, OBF16, W, 1, 64, 2>(a, list, pieces, nnz, st);
    return launch_cfg<BF16, OBF16, W, 1, 64, 4>(a, list, pieces, nnz, st);
}

template <bool BF16, bool OBF16>
static int dispatch(const SpmmArgs &a, bool vec, const ItemList &list, bool pieces, int64_t nnz, hipStream_t st) {
    return a.wt ? dispatch_w<BF16, OBF16, true>(a, vec, list, pieces, nnz, st) : dispatch_w<BF16, OBF16, false>(a, vec, list, pieces, nnz, st);
}

bool spmm_uses_live(const SpOp &op, int F, int64_t ldx) {
    return op.finite_weights && op.ncb == 0 && F > 16 && op.nnz > ROWS_NNZ && op.nnz >= CROWDED_ROW * op.n_in &&
           op.n_in * ldx * 4 >= LIVE_BYTES;
}

int launch_spmm(const SpOp &op, bool restrict_sub, const void *X, int64_t ldx, void *Y, int64_t ldy, int F,
                int dtype, const SpmmEpilogue &ep, hipStream_t stream) {
    int out_dtype = (ep.out_f32 || dtype == CAPGNN_F32) ? CAPGNN_F32 : CAPGNN_BF16;
    if (ep.out_bf16 && dtype == CAPGNN_F32) out_dtype = CAPGNN_BF16;     // float operand, rounded once on the way out
    if (dtype != CAPGNN_F32 && dtype != CAPGNN_BF16) CG_FAIL(CAPGNN_EINVAL, "spmm: unknown dtype %d", dtype);
    if (F <= 0 || F > (1 << 20)) CG_FAIL(CAPGNN_EINVAL, "spmm: F=%d out of range", F);
    if (ldx < F || ldy < F) CG_FAIL(CAPGNN_EINVAL, "spmm: leading dimension smaller than F");
    const int64_t n_rows = restrict_sub ? op.n_sub : op.n_out;
    if (n_rows == 0) return CAPGNN_OK;
    if (!X || !Y) CG_FAIL(CAPGNN_EINVAL, "spmm: NULL operand");
    const int es = elem_bytes(dtype);
    const int ev = 16 / es;
    const int f_up = (F + ev - 1) / ev * ev;
    const int es_out = elem_bytes(out_dtype);
    const bool vec = aligned16(X) && aligned16(Y) && (ldx * es) % 16 == 0 && (ldy * es_out) % 16 == 0 && ldx >= f_up &&
                     ldx * es < (int64_t(1) << 32);
    SpmmArgs a;
    a.idx = op.idx; a.out_scale = op.out_scale;
    a.wt = op.wt;
    if (ep.operand_scaled) {
        if (!op.weights_by_source) CG_FAIL(CAPGNN_EINVAL, "spmm: operand_scaled asks for an operator whose weights depend on the source alone");
        a.wt = nullptr;             // the rows of X carry the weights
    }
    a.items = nullptr; a.n_items = 0; a.n_pieces = 0; a.n_wave = 0;
    a.X = static_cast<const char *>(X); a.ldx_bytes = ldx * es;
    a.Y = static_cast<char *>(Y); a.ldy_bytes = ldy * es_out;
    a.F = F; a.F_lim = vec ? f_up : F;
    a.bias = ep.bias; a.relu = ep.relu;
    a.mask = static_cast<const char *>(ep.mask); a.ldm_bytes = ep.ldm * es_out;
    if (ep.live.bits && dtype == CAPGNN_F32 && spmm_uses_live(op, F, ldx)) a.live = ep.live;
    a.n_in = op.n_in;
    a.acc_rows = ep.accumulate ? static_cast<int>(std::min<int64_t>(ep.acc_rows, INT32_MAX)) : 0;
    if (vec && !restrict_sub && ep.ws) {
        // the blocked kernel runs when the operator has a blocked copy and the caller brought the scratch for it
        const BlockedGeom bg = blocked_geom(op, F, dtype);
        // source offsets are 32-bit counts of 16-byte units formed by a 24-bit multiply
        const bool off_ok = (a.ldx_bytes >> 4) < (int64_t(1) << 24) && op.n_in * (a.ldx_bytes >> 4) < (int64_t(1) << 32);
        if (bg.ok && off_ok && ep.ws_bytes >= bg.ws && (reinterpret_cast<uintptr_t>(ep.ws) & 15u) == 0) {
            float *part = static_cast<float *>(ep.ws);
            if (dtype == CAPGNN_F32 && out_dtype == CAPGNN_BF16) return launch_blocked<false, true>(op, bg, a, part, stream);
            if (dtype == CAPGNN_F32) return launch_blocked<false, false>(op, bg, a, part, stream);
            if (out_dtype == CAPGNN_BF16) return launch_blocked<true, true>(op, bg, a, part, stream);
            return launch_blocked<true, false>(op, bg, a, part, stream);
        }
    }
    // long rows are cut into pieces when the caller brought scratch for their partial sums
    const ItemList &list = restrict_sub ? op.list_sub : op.list;
    a.part = static_cast<float *>(ep.ws); a.ldp = pieces_ldp(F);
    const bool pieces = list.n_cut > 0 && ep.ws && (reinterpret_cast<uintptr_t>(ep.ws) & 15u) == 0 &&
                        ep.ws_bytes >= static_cast<size_t>(list.n_pieces) * a.ldp * sizeof(float);
    if (dtype == CAPGNN_F32 && out_dtype == CAPGNN_BF16) return dispatch<false, true>(a, vec, list, pieces, op.nnz, stream);
    if (dtype == CAPGNN_F32) return dispatch<false, false>(a, vec, list, pieces, op.nnz, stream);
    if (out_dtype == CAPGNN_BF16) return dispatch<true, true>(a, vec, list, pieces, op.nnz, stream);
    return dispatch<true, false>(a, vec, list, pieces, op.nnz, stream);
}

// Measurement aid for the gather roofline: every 8-lane group fetches 128-byte lines (16 bytes per lane) at
// pseudo-random line numbers inside a table, 16 independent loads in flight per lane, nothing else: no index
// stream, no lane exchange, no stores but one checksum per thread.  What it reaches on a table that fits an L2, the
// Infinity Cache, or neither is the rate those levels deliver for this access pattern.
__global__ __launch_bounds__(256) void gather_peak_kernel(const uint4 *table, uint32_t line_mask, uint32_t line_stride, int iters,
                                                          float *out) {
    const uint32_t group = (blockIdx.x * 256u + threadIdx.x) >> 3;
    const uint32_t l = threadIdx.x & 7u;
    const uint4 *base = table + l;
    float acc = 0.f;
    uint32_t x = group * 0x9E3779B1u + 12345u;
    for (int it = 0; it < iters; ++it) {
        uint4 v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            x = x * 1664525u + 1013904223u;                          // the same sequence in all lanes of a group
            const uint32_t line = (x >> 7) & line_mask;              // the high bits of the generator: the low ones cycle
            v[k] = base[static_cast<uint64_t>(line * line_stride) << 3];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)      // all four words are consumed, so the load stays one 16-byte access per lane
            acc += __uint_as_float((v[k].x ^ v[k].y ^ v[k].z ^ v[k].w) & 0x3f800000u);
    }
    out[blockIdx.x * 256u + threadIdx.x] = acc;
}

}  // namespace capgnn

using namespace capgnn;

extern "C" int capgnn_gather_peak(const void *table, int64_t table_lines, int line_stride, int workgroups, int iters,
                                  float *out, double *bytes, void *stream) {
    if (!table || table_lines <= 0 || table_lines > (1LL << 24) || (table_lines & (table_lines - 1)) != 0 || workgroups <= 0 ||
        iters <= 0 || !out || !bytes || !aligned16(table) || line_stride < 1 || table_lines * line_stride > (int64_t(1) << 28))
        CG_FAIL(CAPGNN_EINVAL, "gather_peak: bad argument (table_lines must be a power of two, at most 2^24)");
    hipLaunchKernelGGL(gather_peak_kernel, dim3(workgroups), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const uint4 *>(table), static_cast<uint32_t>(table_lines - 1), static_cast<uint32_t>(line_stride),
                       iters, out);
    CG_HIP(hipGetLastError());
    *bytes = 128.0 * 16.0 * iters * 32.0 * workgroups;      // 32 lane groups per workgroup
    return CAPGNN_OK;
}

extern "C" size_t capgnn_spmm_workspace_bytes(const capgnn_graph *g, int F, int dtype) {
    if (!g || (dtype != CAPGNN_F32 && dtype != CAPGNN_BF16)) return 0;
    return std::max(spmm_ws_bytes(g->fwd, F, dtype), spmm_ws_bytes(g->bwd, F, dtype));
}

extern "C" int capgnn_spmm_fwd(const capgnn_graph *g, const void *X, int64_t ldx, void *Y, int64_t ldy, int F,
                               int dtype, void *ws, size_t ws_bytes, void *stream) {
    if (!g) CG_FAIL(CAPGNN_EINVAL, "spmm_fwd: graph is NULL");
    SpmmEpilogue ep;
    ep.ws = ws; ep.ws_bytes = ws_bytes;
    return launch_spmm(g->fwd, false, X, ldx, Y, ldy, F, dtype, ep, static_cast<hipStream_t>(stream));
}

extern "C" int capgnn_spmm_bwd(const capgnn_graph *g, const void *dY, int64_t lddy, void *dX, int64_t lddx, int F,
                               int dtype, void *ws, size_t ws_bytes, void *stream) {
    if (!g) CG_FAIL(CAPGNN_EINVAL, "spmm_bwd: graph is NULL");
    SpmmEpilogue ep;
    ep.ws = ws; ep.ws_bytes = ws_bytes;
    return launch_spmm(g->bwd, false, dY, lddy, dX, lddx, F, dtype, ep, static_cast<hipStream_t>(stream));
}
