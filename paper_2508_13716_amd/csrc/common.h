// Internal declarations shared by the translation units of libcapgnn (HIP, gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdarg.h>
#include <atomic>
#include <vector>

#include "../../include/capgnn.h"

namespace capgnn {

void set_error(const char *fmt, ...);

#define CG_FAIL(code, ...)                       \
    do {                                         \
        ::capgnn::set_error(__VA_ARGS__);        \
        return (code);                           \
    } while (0)

#define CG_HIP(expr)                                                                     \
    do {                                                                                 \
        hipError_t e__ = (expr);                                                         \
        if (e__ != hipSuccess) {                                                         \
            ::capgnn::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e__),  \
                                __FILE__, __LINE__);                                     \
            return CAPGNN_EHIP;                                                          \
        }                                                                                \
    } while (0)

#define CG_TRY(expr)                 \
    do {                             \
        int rc__ = (expr);           \
        if (rc__ != CAPGNN_OK) return rc__; \
    } while (0)

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline int elem_bytes(int dtype) { return dtype == CAPGNN_BF16 ? 2 : 4; }
static inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// What one lane group of the aggregation kernel walks: a whole short row of the output, or a piece of a long one.
struct alignas(16) RowItem {
    int32_t row;
    uint32_t beg, cnt;          // entries [beg, beg + cnt)
    uint32_t unused;            // one 16-byte load per item
};

// Work list of one direction.  Rows of at least twice `piece` entries are cut into pieces (the last one shorter), whose
// partial sums a second kernel adds in piece order; the pieces come first, then the other rows by entry count,
// descending.  Piece q of cut row k is item piece_first[k] + q.
struct ItemList {
    int64_t n_items = 0, n_pieces = 0, n_cut = 0;
    int64_t max_pieces = 0;                // of one row
    int64_t longest = 0;                   // entries of the longest cut row
    const RowItem *items = nullptr;        // device [n_items]: n_pieces pieces, then whole rows
    const RowItem *cut = nullptr;          // device [n_cut]: the cut rows, whole
    const int32_t *piece_first = nullptr;  // device [n_cut + 1]
    int64_t below[12] = {};                // below[k]: the first item after the pieces that has fewer than 2^k entries

    // the same for the smallest power of two >= entries (at most 2048)
    int64_t first_below(int entries) const {
        int k = 0;
        while (k < 11 && (1 << k) < entries) ++k;
        return below[k];
    }
};

// One direction of the sparse operator: output row k sums over entries [ptr[k], ptr[k+1]).
struct SpOp {
    int64_t n_out = 0;          // rows of the output
    int64_t n_in = 0;           // rows of the gathered operand
    int64_t nnz = 0;
    const int64_t *ptr = nullptr;     // device [n_out+1]
    const int32_t *idx = nullptr;     // device [nnz]   source row of each entry
    // device [nnz]: weight of each entry, edge value * in_scale[source] formed once (a sequential read in the
    // kernels instead of a gather from in_scale per entry); null when every weight is 1
    const float *wt = nullptr;
    // no edge values: the weight of an entry is in_scale[source] alone, so a caller that multiplies row s of the
    // operand by in_scale[s] first may ask for the unweighted sum (SpmmEpilogue::operand_scaled)
    bool weights_by_source = false;
    bool finite_weights = false;      // no weight is infinite or NaN: an all-zero row adds nothing, whatever its weight
    const float *out_scale = nullptr; // device [n_out] or null
    const float *in_scale = nullptr;  // device [n_in]  or null
    // output rows by entry count, descending; rows shorter than EXACT_ROW only by power-of-two class, in index order
    // inside a class
    const int32_t *order = nullptr;   // device [n_out]
    int64_t n_sub = 0;                // rows [0, n_sub) of the output: the restricted list (bwd: local columns only)
    ItemList list, list_sub;          // of all output rows, and of the restricted ones
    // Column-blocked copy of the entries (built for dense-degree operators whose gathered operand does not
    // fit an L2): entries regrouped by (source block cb = idx / CB_ROWS, position p in `order`), original
    // entry order kept inside a group.  Group (cb, p) = entries [b_off[cb*n_out+p], b_off[cb*n_out+p+1]).
    int ncb = 0;                      // 0: no blocked copy
    const uint32_t *b_off = nullptr;  // device [ncb*n_out + 1]
    const int2 *b_ew = nullptr;       // device [nnz]  {source row, bits of the float weight val * in_scale[source]}
    // the same entries without their weights, as 16-bit row numbers inside the block (operators without edge values): read instead of b_ew when
    // every weight is 1, or when the caller has multiplied the operand rows by in_scale beforehand
    const uint16_t *b_src = nullptr;  // device [nnz] or null: source row - cb * CB_ROWS (2 bytes per entry)
    // positions [0, b_long) hold rows whose groups are long enough for a whole workgroup, [b_long, b_mid) for
    // one wave per group, the rest are walked eight rows per wave (`order` is descending in entry count)
    int64_t b_long = 0, b_mid = 0;
};

constexpr int EXACT_ROW = 256;  // work lists sort rows at least this long by their exact entry count
constexpr int CB_ROWS = 32768;  // source rows per column block: 32768 x 128-byte slices = 4 MB, one XCD's L2 (swept: 8192 .. 49152)
constexpr int B_LONG_GROUP = 1024; // rows with at least this many entries per source block on average: workgroup per group (swept 256 .. 4096)
constexpr int B_MID_GROUP = 256;  // ... at least this many: wave per group (swept 64 .. 1024; the eight-rows-per-wave class below is the fastest)
constexpr int SLICE_BYTES = 128;  // feature bytes of one source row that one task of the blocked kernel gathers
constexpr int NUM_CU = 256;       // compute units of the chip
constexpr int NUM_XCD = 8;        // L2 domains of the chip; workgroup b is dispatched to domain b % NUM_XCD

}  // namespace capgnn

struct capgnn_graph {
    int64_t n_loc = 0, n_halo = 0, n_cols = 0, nnz = 0;
    uint32_t flags = 0;
    capgnn::SpOp fwd, bwd;
    std::vector<void *> dev_allocs;
    // pinned words in which an epoch's last kernel leaves the loss for the host, one cache line per epoch under way (bit i of `taken`: line i)
    static constexpr int LOSS_LINES = 16, LOSS_STRIDE = 32;
    float *loss_host = nullptr, *loss_dev = nullptr;
    mutable std::atomic<unsigned> taken{0};
};

struct capgnn_cache {
    int64_t n_halo = 0, cap_gpu = 0, n_host = 0;
    int n_layers = 0, dtype = 0, map_kind = 0;
    std::vector<int32_t> dims;
    std::vector<int64_t> pitch;         // row pitch in bytes per layer
    std::vector<size_t> gpu_off, host_off;  // byte offset of each layer's table inside the tiers
    char *gpu_tier = nullptr;
    char *host_tier = nullptr;
    // host copies
    std::vector<int32_t> slot_h;        // [n_halo]  >=0: GPU slot, <0: host slot = -1-value
    std::vector<int64_t> gid_h;
    std::vector<int64_t> hkeys_h;       // hash table keys (gid) ...
    std::vector<int32_t> hvals_h;       // ... and halo-local index, -1 = empty
    uint64_t hmask = 0;
    // device copies
    int32_t *slot_d = nullptr;
    int32_t *gpu_list_d = nullptr;      // [cap_gpu]  halo-local index of GPU slot k
    int32_t *host_list_d = nullptr;     // [n_host]
    int64_t *hkeys_d = nullptr;
    int32_t *hvals_d = nullptr;
    int64_t *counters_d = nullptr;      // [4] hits, misses, absent
    int64_t *stamp_d = nullptr;         // [n_layers][n_halo] iteration in which each cached row was last written
    long long *owner_d = nullptr;       // [n_halo] scratch of an update call: position of the last update of a vertex
    int64_t *scan_d = nullptr;          // [n_halo/1024 + 2] scratch of the stale-list compaction
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    std::vector<hipEvent_t> ev_layer;   // one per layer: host-tier rows of that layer have landed
    std::vector<hipEvent_t> ev_consumed;  // one per layer: the layer's staging area has been scattered (pipelined mode)
    std::vector<uint8_t> staged_valid;  // pipelined mode: staging area of layer l holds rows copied for the next epoch
    void *staged_base = nullptr;        // ... inside this staging area
    hipStream_t last_side = nullptr;    // stream that may still carry such a copy
    int miss_mode = CAPGNN_MISS_STAGED;
    std::vector<void *> dev_allocs;
};

namespace capgnn {

// Which rows of a matrix may differ from zero: row r if bit r % 32 of bits[r / 32] is set (whole words of 32 rows, the rest of the
// last one unset or not there), *count of them in all; both on the device.  No bits: any row.
struct LiveRows {
    const uint32_t *bits = nullptr;
    const float *count = nullptr;
};

// ---- kernels' host-side launchers (each validates what its kernel assumes) ----
// What is left to add up at the end of an epoch, and the SGD step, for one launch (see epoch_finish_kernel in ops.hip).
struct FinishTask {
    enum Kind : int { SUM, COLUMNS, LOSS_COLUMNS, LOSS, UPDATE };
    int kind, S;                // S partial results ...
    int64_t n;                  // ... of n numbers each
    const void *part;           // [S][n] float; LOSS: [S] double, UPDATE: [n] float, the gradient
    float *out, *out2;          // their sums; LOSS: the loss, and where else it goes, or null
    float *W;                   // W -= lr * sum, or null
    const float *norm_dev;      // LOSS: the normaliser (norm_dev, or norm_val where that is null)
    float norm_val;
    unsigned first;             // filled by launch_finish
};
struct FinishList {
    static constexpr int MOST = 48;
    FinishTask task[MOST];
    int count = 0;
    bool full() const { return count >= MOST; }
};
// lr != 0: also the tensors of `sgd`, in their order where some share memory
struct SgdList;
int launch_finish(FinishList *list, const SgdList *sgd, float lr, hipStream_t stream);

struct SpmmEpilogue {
    const float *bias = nullptr;   // [F] added after scaling
    int relu = 0;
    int accumulate = 0;            // add the previous contents of Y
    int64_t acc_rows = INT64_MAX;  // ... in output rows below this one
    const void *mask = nullptr;    // [rows x ldm] of Y's storage type: Y is zeroed where it is not positive
    int64_t ldm = 0;
    int out_f32 = 0;               // store Y as float although X is bf16
    int out_bf16 = 0;              // store Y as bf16 although X is float (the loss gradient of a bf16 model is gathered unrounded)
    LiveRows live;                 // rows of X that need not be read, being zero throughout
    int operand_scaled = 0;        // row s of X already carries in_scale[s] (only for operators with weights_by_source)
    void *ws = nullptr;            // scratch for the column-blocked kernel or for cut rows (spmm_ws_bytes), may be null
    size_t ws_bytes = 0;
};

size_t spmm_ws_bytes(const SpOp &op, int F, int dtype);

// whether an aggregation of float rows (F elements at a pitch of ldx) makes use of SpmmEpilogue::live
bool spmm_uses_live(const SpOp &op, int F, int64_t ldx);

int launch_spmm(const SpOp &op, bool restrict_sub, const void *X, int64_t ldx, void *Y, int64_t ldy, int F,
                int dtype, const SpmmEpilogue &ep, hipStream_t stream);

// Products that do not wait for one another, collected between begin (the calling thread's batch, emptied) and launch (gemm.hip)
struct SmallBatch;
SmallBatch *small_batch_begin();
int launch_small_batch(SmallBatch *b, hipStream_t stream);

int launch_gemm(int trans_a, int trans_b, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
                const void *B, int64_t ldb, void *C, int64_t ldc, int dtype, int out_f32, int accumulate,
                const float *bias, int relu, const void *relu_mask, int64_t ldm, void *ws, size_t ws_bytes,
                hipStream_t stream, const float *row_scale = nullptr,    // row_scale: C[i,:] *= row_scale[i] at the very end (fp32 C)
                int f32_product = CAPGNN_F32_PRODUCT_AUTO,
                float *colsum = nullptr,                                 // [N] column sums of B (trans_a && !trans_b only)
                FinishList *later = nullptr,                             // takes the sum over splits, whose parts stay in ws, if it can
                SmallBatch *batch = nullptr);                            // may take the product: it runs with launch_small_batch
// C = A op(W) + A2 op(W2) (+ bias, ReLU), one launch where a kernel forms the sum, else the two launches it replaces
int launch_gemm_dual(int trans_b, int64_t M, int64_t N, int64_t K1, const void *A, int64_t lda, const void *W, int64_t ldw, int64_t K2,
                     const void *A2, int64_t lda2, const void *W2, int64_t ldw2, void *C, int64_t ldc, int dtype, int out_f32,
                     const float *bias, int relu, void *ws, size_t ws_bytes, hipStream_t stream, int f32_product,
                     const void *relu_mask = nullptr, int64_t ldm = 0, SmallBatch *batch = nullptr);
// C = op(A) op(B) (rows scaled) and C2 = op(A2) op(B2), one launch for small and middling sizes
int launch_gemm_pair(int trans_a, int trans_b, int64_t M, int64_t M2, int64_t N, int64_t K, const void *A, int64_t lda, const void *A2,
                     int64_t lda2, const void *B, int64_t ldb, const void *B2, int64_t ldb2, void *C, int64_t ldc, void *C2,
                     int64_t ldc2, int dtype, int out_f32, const float *row_scale, void *ws, size_t ws_bytes, hipStream_t stream,
                     int f32_product, float *colsum = nullptr, FinishList *later = nullptr, SmallBatch *batch = nullptr);
size_t gemm_pair_ws_bytes(int trans_a, int64_t M, int64_t N, int64_t K);
// scratch that lets launch_gemm_dual run as one launch
size_t gemm_dual_ws_bytes(int64_t N, int64_t K1, int64_t K2);
size_t gemm_ws_bytes(int trans_a, int64_t M, int64_t N, int64_t K);

// dZ = dH * 1[H > 0] in place (when relu) and dbias[f] = sum_i dZ[i,f] (when dbias), fixed summation order.
// src (of src_dtype, pitch lds), when non-null and different from dH, is the unrounded gradient: dH is then
// written as its masked, converted copy and the bias gradient is summed from the unrounded values.
size_t relu_bias_ws_bytes(int64_t n, int F);
int launch_relu_mask_dbias(int64_t n, int F, const void *src, int64_t lds, int src_dtype, void *dH, int64_t lddh,
                           const void *H, int64_t ldh, int dtype, int h_dtype, int relu, float *dbias, void *ws,
                           size_t ws_bytes, hipStream_t stream, const float *row_scale = nullptr);
// tensors of one SGD step (three per layer at most), in the order in which they are updated
struct SgdList {
    float *W[48];
    const float *dW[48];
    int64_t n[48];
    unsigned first[48];         // filled by launch_sgd
    int count = 0;
};
int launch_sgd(const SgdList &all, float lr, hipStream_t stream);
// the loss of an epoch on labels or targets, with what else can be had on the way (see ops.hip)
int loss_epoch(int64_t n, int C, const float *Z, int64_t ldz, const int32_t *labels, const uint8_t *targets, int64_t ldt,
               const uint8_t *mask, double loss_norm, float *loss_dev, void *dZ, int64_t lddz, int dz_dtype, float *copy, float *dbias,
               const float *row_scale, LiveRows *live, void *ws, size_t ws_bytes, hipStream_t st, FinishList *later = nullptr);
size_t loss_epoch_ws_bytes(int64_t n, int C);
bool loss_sums_columns(int C);      // whether loss_epoch can form dbias

uint64_t hash_gid(uint64_t x);

// full-batch gather of one layer's halo rows, one tier at a time (used by the epoch's two-stream schedule)
int gather_all_hits(const capgnn_cache *c, int layer, void *out, int64_t ld, hipStream_t st);
// the same for the first L layers in one launch, where that is a few small copies; *done says whether it was
int gather_all_hits_of_layers(const capgnn_cache *c, int L, char *const *out, const int64_t *ld, hipStream_t st, bool *done);
int gather_all_misses(const capgnn_cache *c, int layer, void *out, int64_t ld, void *staging, hipStream_t st);
// the two halves of the staged path: DMA of the layer's host tier into the staging area, scatter from there
int stage_misses(const capgnn_cache *c, int layer, void *staging, hipStream_t st);
int scatter_staged(const capgnn_cache *c, int layer, void *out, int64_t ld, void *staging, hipStream_t st);
int gather_hits_and_staged(const capgnn_cache *c, int layer, void *out, int64_t ld, void *staging, hipStream_t st);

}  // namespace capgnn
