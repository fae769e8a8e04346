// Internal helpers shared by the HIP translation units of libgrappa_hip.so.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <functional>
#include <vector>
#include <hip/hip_bf16.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>

#include "../../include/grappa.h"

namespace grp {

// ---------------------------------------------------------------- errors
void set_error(const char* fmt, ...);
grp_status fail(grp_status code, const char* fmt, ...);

#define GRP_HIP(call)                                                                   \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            return grp::fail(GRP_EHIP, "%s failed: %s (%s:%d)", #call,                  \
                             hipGetErrorString(e_), __FILE__, __LINE__);                \
    } while (0)

#define GRP_TRY(call)                                                                   \
    do {                                                                                \
        grp_status s_ = (call);                                                         \
        if (s_ != GRP_OK) return s_;                                                    \
    } while (0)

// ---------------------------------------------------------------- profiling
// Brackets a kernel launch with two events when profiling is enabled.
// flops / bytes: the algorithmic work of the launch (what the operation must compute and
// move, not what the kernel happens to touch); summed per kernel name in the report.
void prof_begin(const char* name, hipStream_t st, double flops, double bytes);
void prof_end(hipStream_t st);
// Optional shape suffix for the next prof_begin on this thread (only with profile mode 2).
void prof_detail(const char* fmt, ...);

struct ProfScope {
    hipStream_t st;
    ProfScope(const char* name, hipStream_t s, double flops = 0.0, double bytes = 0.0) : st(s) {
        prof_begin(name, s, flops, bytes);
    }
    ~ProfScope() { prof_end(st); }
};

// Checks the launch itself (bad configuration etc.); kernels run asynchronously.
#define GRP_LAUNCH_CHECK()                                                              \
    do {                                                                                \
        hipError_t e_ = hipGetLastError();                                              \
        if (e_ != hipSuccess)                                                           \
            return grp::fail(GRP_EHIP, "kernel launch failed: %s (%s:%d)",              \
                             hipGetErrorString(e_), __FILE__, __LINE__);                \
    } while (0)

}  // namespace grp

// ---------------------------------------------------------------- launches of several steps merged
// A launch costs the device about 3.6 us whatever it does, and the steps of a phase's partitions are the same launches on other data.
// (Four steps of 2 500 nodes, GCN 64-64-8: some 100 launches and 427 us one after another, 28 and 145 us merged; separate streams do not help:
// launches of different queues cost the same 3.6 us each.)
// grp_train_steps lets every step record its launches instead of making them, and then makes one launch of those that are the same
// kernel at the same point of their steps: blockIdx.z says whose arguments a workgroup takes.
//
// A kernel takes part through three things: its body as a device function whose first parameter is the step's own gridDim.x, the kernel
// around it, and an Op that names the body:  struct Op { static constexpr int THREADS, WGS; template <class... A> static
// __device__ void run(unsigned gx, const A&... a) { body(gx, a...); } }.  launch(kernel, Op(), ...) then does either.
namespace grp {

template <class... P> struct Pack {};
template <class H, class... T> struct Pack<H, T...> { H head; Pack<T...> tail; };
template <class... P> struct Packer { static Pack<> make() { return {}; } };
template <class H, class... T> struct Packer<H, T...> {
    static Pack<H, T...> make(H h, T... t) { return Pack<H, T...>{h, Packer<T...>::make(t...)}; }
};
template <class Op, class... A> __device__ __forceinline__ void unpack(unsigned gx, const Pack<>&, const A&... a) { Op::run(gx, a...); }
template <class Op, class H, class... T, class... A>
__device__ __forceinline__ void unpack(unsigned gx, const Pack<H, T...>& p, const A&... a) { unpack<Op>(gx, p.tail, a..., p.head); }

constexpr size_t MANY_ARG_BYTES = 3584;            // of the 4 KB that a launch's arguments may take
constexpr int MANY_MOST = 8;
template <class P> constexpr int many_of() {
    return MANY_ARG_BYTES / (sizeof(P) + 4) >= MANY_MOST ? MANY_MOST : (int)(MANY_ARG_BYTES / (sizeof(P) + 4));
}
template <class P> struct Many {
    P at[many_of<P>() > 0 ? many_of<P>() : 1];
    uint32_t gx[many_of<P>() > 0 ? many_of<P>() : 1];
};
template <class Op, class P> __global__ __launch_bounds__(Op::THREADS, Op::WGS) void many_kernel(Many<P> m) {
    const uint32_t gx = m.gx[blockIdx.z];
    if (blockIdx.x < gx) unpack<Op>(gx, m.at[blockIdx.z]);
}

struct LaunchRecord {
    void (*go)(const LaunchRecord* const* recs, int count, hipStream_t st) = nullptr;     // launches `count` records of this kind (the same go)
    dim3 grid;
    std::vector<unsigned char> args;               // a Pack
    std::function<void()> alone;                   // a launch that is not merged (go: null)
};
struct LaunchRecorder {
    std::vector<LaunchRecord> list;
    bool refused = false;                          // a launch that no merged step has was asked for (and not made)
    int steps = 1;                                 // that may share a launch
};
extern thread_local LaunchRecorder* g_recorder;    // null: launches are made at once

template <class Op, class P> void launch_many(const LaunchRecord* const* recs, int count, hipStream_t st) {
    constexpr int N = many_of<P>();
    static_assert(N > 0, "the arguments of one step must fit a launch");
    for (int i0 = 0; i0 < count; i0 += N) {
        const int n = count - i0 < N ? count - i0 : N;
        Many<P> m;
        memset((void*)&m, 0, sizeof m);
        dim3 grid(1, 1, (unsigned)n);
        for (int i = 0; i < n; ++i) {
            const LaunchRecord& r = *recs[i0 + i];
            memcpy((void*)&m.at[i], r.args.data(), sizeof(P));
            m.gx[i] = r.grid.x;
            grid.x = std::max(grid.x, r.grid.x);
            grid.y = r.grid.y;                     // (alike: launch_merged)
        }
        hipLaunchKernelGGL((many_kernel<Op, P>), grid, dim3(Op::THREADS), 0, st, m);
    }
}

// One launch, made or recorded (no dynamic LDS, one thread count: Op::THREADS).
template <class Op, class... P, class... A> void launch(void (*kernel)(P...), Op, dim3 grid, hipStream_t st, A... a) {
    if (!g_recorder) {
        hipLaunchKernelGGL(kernel, grid, dim3(Op::THREADS), 0, st, P(a)...);
        return;
    }
    const Pack<P...> p = Packer<P...>::make(P(a)...);
    g_recorder->list.emplace_back();
    LaunchRecord& r = g_recorder->list.back();
    r.go = &launch_many<Op, Pack<P...>>;
    r.grid = grid;
    r.args.assign((const unsigned char*)&p, (const unsigned char*)&p + sizeof p);
}
// The same of a kernel without an Op, which steps that are otherwise merged launch one by one: what few models or odd sizes run.
template <class... P, class... A> void launch_alone(void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t st, A... a) {
    if (!g_recorder) {
        hipLaunchKernelGGL(kernel, grid, block, lds, st, P(a)...);
        return;
    }
    g_recorder->list.emplace_back();
    g_recorder->list.back().alone = [=] { hipLaunchKernelGGL(kernel, grid, block, lds, st, P(a)...); };
}
// In front of a launch that is large by itself: false if it must not be made, because launches are being recorded (such steps are made one
// by one: their launches do not bound them, and side by side they would take the caches from each other).
inline bool may_launch() {
    if (g_recorder) g_recorder->refused = true;
    return !g_recorder;
}
#define GRP_LARGE_LAUNCH(...) do { if (grp::may_launch()) hipLaunchKernelGGL(__VA_ARGS__); } while (0)

}  // namespace grp

namespace grp {
// ---------------------------------------------------------------- device memory of the builders (runtime.hip)
// As hipMalloc / hipFree, from a bounded cache of freed blocks.
hipError_t pool_alloc(void** p, size_t bytes);
void pool_free(void* p);
hipError_t pool_release();         // gives back what is kept on the current device

// ---------------------------------------------------------------- partition handle
}  // namespace grp

namespace grp {
// Rows longer than SPMM_LONG_ROW edges are cut into chunks of at most SPMM_CHUNK edges
// (device arrays, built once with the partition; see spmm.hip).
constexpr int SPMM_LONG_ROW = 128;
constexpr int SPMM_CHUNK = 512;
// Source-sliced schedule of the long rows of a large structure (slices.hip): a long row is cut where its
// sorted sources cross from one of SLICES equal ranges of node ids into the next, and each segment into tasks
// of at most SLICE_TASK_MAX edges; the tasks are processed slice by slice.
constexpr int SLICES = 64;
constexpr int SLICE_PIECE = 128;       // edges a wavefront takes in one pass (two indices per lane)
constexpr int SLICE_TASK_MAX = 1024;   // edges of a task: up to this many consecutive edges of one piece share a partial row
                                       // (128, i.e. a partial row per pass: 40 % more partial rows, step 142.3 against 139.0 ms; 4096: 139.7)
constexpr int SLICE_MIN_PIECE = 112; // a row is not cut at a slice boundary before its current piece has this many edges
                                     // (measured on the 2^32-edge share, ms per step: 64: 153.3 and 96: 145.5 with tasks of at most 128
                                     //  edges; with tasks of up to 1024: 80: 143.1, 96: 139.0, 112: 137.3, 128: 137.6, 144: 137.6; the
                                     //  10^8-edge share with 1 KB rows prefers shorter pieces: 96: 291, 112: 295, 128: 297 ms per step)
struct SliceTask {
    int64_t begin;                   // first edge of the task
    uint32_t id;                     // its number in row-major order: where its partial row goes
    uint32_t len;                    // 1 .. SLICE_TASK_MAX edges
};
struct LongRows {
    int32_t n_long = 0, n_chunks = 0;
    int32_t* long_row = nullptr;     // [n_long]    row index
    int32_t* long_first = nullptr;   // [n_long+1]  first chunk of each long row
    int64_t* chunk_begin = nullptr;  // [n_chunks]  edge range of the chunk
    int64_t* chunk_end = nullptr;    // [n_chunks]
    // the sliced schedule of the same rows (n_tasks = 0: not built; the aggregation then walks the chunks)
    int64_t n_tasks = 0;
    SliceTask* tasks = nullptr;      // [n_tasks] in processing order (slice-major, rows ascending inside a slice)
    int64_t* row_task = nullptr;     // [n_long+1] first task id of each long row
};
}  // namespace grp

struct grp_partition_s {
    grp::LongRows csr_long, csc_long;
    int64_t n = 0, nnz = 0;
    int64_t* l2g = nullptr;
    int64_t* rowptr = nullptr;
    int32_t* col = nullptr;
    int64_t* colptr = nullptr;
    int32_t* row = nullptr;
    int32_t* d_local_in = nullptr;
    int32_t* d_local_out = nullptr;
    int64_t* d_global_in = nullptr;
    // weighted partitions only (null otherwise): edge weights in CSR / CSC order and the weight
    // masses of every node's local / global in-edges
    float* csr_w = nullptr;
    float* csc_w = nullptr;
    double* w_local_in = nullptr;
    double* w_global_in = nullptr;
    uint8_t* base_mask = nullptr;    // partitions built from chunks: 1 for the base chunk's nodes
    void* slab = nullptr;            // one allocation that holds the CSR / CSC arrays and the long-row schedules
    size_t slab_bytes = 0;
    bool borrowed_csr = false;       // rowptr / col belong to the caller (grp_partition_from_csr): never freed here
    int device = 0;
};

// The graph split once into chunks: edges grouped by (chunk(dst), chunk(src)) so that the
// partition base + swept reads only its four groups, and the global in-degree of every node.
struct grp_chunks_s {
    int32_t n_chunks = 0;
    uint64_t seed = 0;
    int64_t N = 0, E = 0;
    int64_t* src = nullptr;          // [E] global ids, grouped by bucket (order inside a bucket arbitrary)
    int64_t* dst = nullptr;
    int64_t* d_global_all = nullptr; // [N]
    int32_t* assign = nullptr;       // [N] caller-supplied chunk of every node (null: the random split by seed)
    std::vector<int64_t> bucket_ptr; // host, [n_chunks^2 + 1], bucket = chunk(dst) * n_chunks + chunk(src)
    int device = 0;
};

namespace grp {

// The sliced schedules of the handle's long rows, where they pay (slices.hip).  long_edges: the edges of each direction's long rows
// (negative: counted there).
grp_status build_slice_tasks(grp_partition_t* h, const int64_t (&long_edges)[2], hipStream_t st);

// Exclusive prefix sum over a workgroup of WAVES full wavefronts; total: of all.  Starts on a barrier.
template <int WAVES, typename T> __device__ __forceinline__ T block_scan(T v, T* wave_sum /*[WAVES], LDS*/, T& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    __syncthreads();
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    T before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w < wave) before += wave_sum[w];
        all += wave_sum[w];
    }
    total = all;
    return before + incl - v;
}

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }

// add(load(c), true) for c in [c0, c1), in this order, eight loads in flight, four at the end: a place past the end is loaded from the last
// one again and handed over with false.  (Loaded one by one, the longest row's partial rows were what the launches that combine them waited for:
// 3e5 rows of 256, sums 9.1 -> 5.5 us, attention 10.1 -> 5.6; 1e5 rows of 75 7.1 -> 4.9.)
template <class Load, class Add> __device__ __forceinline__ void in_order(int c0, int c1, Load load, Add add) {
    typedef decltype(load(0)) T;
    int c = c0;
    for (; c + 8 <= c1; c += 8) {
        T v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = load(c + u);
#pragma unroll
        for (int u = 0; u < 8; ++u) add(v[u], true);
    }
    for (; c < c1; c += 4) {
        T v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = load(imin(c + u, c1 - 1));
#pragma unroll
        for (int u = 0; u < 4; ++u) add(v[u], c + u < c1);
    }
}

// 16 and 8 bytes at any element boundary: global loads of these need no alignment beyond the element's
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(2)));

typedef uint32_t u32x4_al __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_al __attribute__((ext_vector_type(2)));

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline int64_t round_up(int64_t a, int64_t b) { return cdiv(a, b) * b; }

// ---------------------------------------------------------------- kernels (host launchers)
// Neighbour aggregation over a CSR-like structure (ptr/idx), one output row per group of
// lanes.  Y[i,:] = a_i (sum_e X[idx[e],:] + self*X[i,:]) (+ addend[i,:]) (+ bias) (ReLU).
struct SpmmArgs {
    const int64_t* ptr = nullptr;   // [n_rows+1]
    const int32_t* idx = nullptr;   // [nnz]
    int64_t nnz = 0;                // (with n_rows, what chooses between kernels)
    int64_t n_src = 0;              // rows of X, above every idx (0 = n_rows): some kernels read rows beyond it as zeros
    int64_t n_rows = 0;
    int32_t F = 0;
    const void* X = nullptr;
    int64_t ldx = 0;
    int32_t x_bf16 = 0;
    int32_t scale = GRP_SCALE_NONE;
    int32_t self_term = 0;
    const float* colscale = nullptr;  // per gathered row multiplier [n_src] or null
    const float* addend = nullptr;  // [n_rows x F] or null (may alias Y)
    int64_t ld_add = 0;
    const float* bias = nullptr;    // [F] or null
    int32_t relu = 0;
    float* Y = nullptr;
    int64_t ldy = 0;
    const LongRows* long_rows = nullptr;  // null = no row is split
    float* partials = nullptr;            // [n_chunks x round_up(F,4)] scratch when rows are split
    int64_t addend_rows = 0;              // rows >= this have no addend (0: every row has one)
    const float* mask = nullptr;          // result kept where mask[i,c] > 0, else 0 (after the ReLU)
    int64_t ld_mask = 0;
    const float* residual = nullptr;      // added after the ReLU: Y = residual + act (residual layers)
    int64_t ld_res = 0;
    float* Y2 = nullptr;                  // also receives act (before the residual is added)
    int64_t ldy2 = 0;
    const float* val = nullptr;           // [nnz] per-edge multiplier of the gathered row, or null
    const float* rowscale = nullptr;      // [n_rows] a_i given explicitly (replaces `scale`), or null
    // Sizes known on the device only (blocks sampled without a host round trip).  When set, n_rows and
    // addend_rows above are upper bounds that size the launch (ptr must be valid, with empty rows, up to
    // n_rows) and the kernels stop at the values stored here.
    const int64_t* n_rows_dev = nullptr;
    const int64_t* addend_rows_dev = nullptr;
};
grp_status launch_spmm(const SpmmArgs& a, hipStream_t st);
size_t spmm_partials_bytes(const LongRows* lr, int32_t F);

struct StepSums;

// C[M x N] = epilogue(A[M x K] B[K x N] + A2[M x K2] B2[K2 x N])
// epilogue: (+ bias[N]) (+ addend[M x N]) (* rowscale[M]) (ReLU) (* (mask[M x N] > 0))
struct GemmNNArgs {
    int64_t M = 0;
    int32_t N = 0, K = 0;
    const void* A = nullptr;
    int64_t lda = 0;
    int32_t a_bf16 = 0;
    const float* B = nullptr;
    int64_t ldb = 0;
    int32_t K2 = 0;                 // 0 = no second product
    const float* A2 = nullptr;
    int64_t lda2 = 0;
    const float* B2 = nullptr;
    int64_t ldb2 = 0;
    const float* bias = nullptr;
    const float* addend = nullptr;
    int64_t ld_add = 0;
    const float* rowscale = nullptr;
    int32_t relu = 0;
    const float* mask = nullptr;
    int64_t ld_mask = 0;
    float* C = nullptr;
    int64_t ldc = 0;
    int32_t zero_pad_to = 0;        // also write zeros to columns [N, zero_pad_to)
    const int32_t* a_rows = nullptr; // row i of A is stored at row a_rows[i] (null: i)
    int64_t a_valid_rows = 0;       // rows >= this of the FIRST product's A read as zero (0: M)
    float* C_raw = nullptr;         // also receives acc + bias + addend (before scale / ReLU / mask)
    int64_t ld_raw = 0;
    int32_t rowscale_cols = 0;      // rowscale applies to columns < this only (0: all columns)
    int32_t bias_col0 = 0;          // bias[c - bias_col0] is added to columns c in [bias_col0, bias_col0 + bias_n)
    int32_t bias_n = 0;             // (0: N - bias_col0)
    int32_t a_tight = 0;            // set by the launch: rows of A end at column K or are not 16-byte friendly
    const float* Bt = nullptr;      // when set: B given transposed, Bt[N x K] (pitch ldbt), fast path
    int64_t ldbt = 0;
    const float* Bt2 = nullptr;     // same for the second product
    int64_t ldbt2 = 0;
    // Bt and Bt2 as planes that exist already (bt_planes_at), of ready_rows rows each, or null: then, if set, `planes` is scratch of
    // gemm_planes_bytes for them to be made once per launch.  (Set by the launch too: what the kernel reads.)
    const unsigned char *ready = nullptr, *ready2 = nullptr;
    int32_t ready_rows = 0;
    unsigned char* planes = nullptr;
    size_t planes_bytes = 0;
    // Row counts known on the device only: when set, M (and a_valid_rows) above are upper bounds that
    // size the launch, and the kernels read the real values here.
    const int64_t* M_dev = nullptr;
    const int64_t* a_valid_rows_dev = nullptr;
    // When set: also the column sums of C, row m times col_mul[m], to col_out[N] through `sums`, by way of col_part (a row of N floats for
    // every 64 rows of C).  For fp32 A of whole 16-byte units, all rows valid, and ready planes.
    StepSums* sums = nullptr;
    float *col_part = nullptr, *col_out = nullptr;
    const float* col_mul = nullptr;
};
size_t gemm_planes_bytes(int64_t M, int32_t N, int32_t K);      // K: of both products together
grp_status launch_gemm_nn(const GemmNNArgs& a, hipStream_t st);

// Partial statistics of a step's loss rows.
struct StatsPartial {
    double ratio, r_dbl;
    int64_t s, r_int;
};

struct NnzParts {
    const int64_t* p[GRP_MAX_LAYERS];
    int n;
    const int64_t* bad_seeds;      // null, or the number of seeds that were outside the partition
};

// What a step's record is made of.
struct RecordArgs {
    const StatsPartial* part;
    int blocks, full_graph;
    int64_t nnz_const;
    NnzParts np;
    const double* loss_part;
    int loss_blocks;
    grp_step_stats* out;
};

// Sums over partial results that nothing but a step's gradient waits for, done by its last launch together with its record
// (a mini-batch step of three layers makes 32 launches; 36 with a launch for each).
enum SumKind : uint8_t { SUM_TN, SUM_TN_4WAY, SUM_TN_VEC, SUM_COLUMNS };
constexpr int64_t sum_block(SumKind kind) { return kind == SUM_TN ? 256 : kind == SUM_COLUMNS ? 8 : 64; }      // elements of a workgroup
constexpr uint32_t NO_SUM = ~0u;
struct SumJob {
    uint32_t part;                   // units of 16 bytes of the workspace
    uint32_t C, C2, colsum;          // elements of the gradient (NO_SUM: none)
    uint32_t begin;                  // its first workgroup
    int32_t count;                   // partial results
    uint16_t K, N;
    uint8_t dual, kind;
};
template <int MOST> struct StepSumsOf {
    const char* base = nullptr;      // the workspace
    float* grad = nullptr;
    RecordArgs record = {};
    uint32_t record_blocks = 0;      // 1: there is a record to be made
    int32_t n = 0;
    SumJob job[MOST];
};
constexpr int STEP_SUMS = 3 * GRP_MAX_LAYERS;
struct StepSums : StepSumsOf<STEP_SUMS> {
    uint32_t blocks = 0;
    double bytes = 0.0;
    StepSums(const void* workspace, float* gradient) { base = (const char*)workspace; grad = gradient; }
    // elements: that the sums give
    void add(SumKind kind, const void* part, int32_t count, int32_t K, int32_t N, int dual, const float* C, const float* C2, const float* colsum,
             int64_t elements) {
        auto at = [&](const float* p) { return p ? (uint32_t)(p - grad) : NO_SUM; };
        job[n++] = SumJob{(uint32_t)(((const char*)part - base) / 16), at(C), at(C2), at(colsum), blocks, count, (uint16_t)K, (uint16_t)N, (uint8_t)dual,
                          (uint8_t)kind};
        blocks += (uint32_t)cdiv(elements, sum_block(kind));
        bytes += 4.0 * (double)elements * (count + 1.0);
    }
};
grp_status launch_step_sums(const StepSums& s, hipStream_t st);

// C[K x N] = A[M x K]^T B[M x N], fixed-order split over M.
size_t gemm_tn_workspace_bytes(int64_t M, int32_t K, int32_t N);
struct GemmTNArgs {
    int64_t M = 0;
    int32_t K = 0, N = 0;
    const void* A = nullptr;
    int64_t lda = 0;
    int32_t a_bf16 = 0;
    const float* B = nullptr;
    int64_t ldb = 0;
    float* C = nullptr;
    int64_t ldc = 0;
    void* workspace = nullptr;
    size_t workspace_bytes = 0;
    const int32_t* a_rows = nullptr; // row i of A is stored at row a_rows[i] (null: i)
    float* colsum_out = nullptr;     // optional [N]: column sums of B
    // A second product from the same launch (at most one of the two):
    const float* A2 = nullptr;       // C2[K x N] = A2[M x K]^T B   (fp32, rows not gathered)
    int64_t lda2 = 0;
    const float* B2 = nullptr;       // C2[K x N] = A^T B2[M x N]
    int64_t ldb2 = 0;
    float* C2 = nullptr;             // pitch ldc
    const int64_t* M_dev = nullptr;  // when set: the real number of rows (on the device); M above is an upper bound
    int32_t a_tight = 0, b_tight = 0;    // set by the launch: rows of A / B end at their last column or are not 16-byte friendly
    StepSums* sums = nullptr;        // when set (and ldc = N): the sum over the slices is left to it, the workspace is in use until then
};
grp_status launch_gemm_tn(const GemmTNArgs& a, hipStream_t st);

// out[N] = column sums of A[M x N], every row multiplied by rowmul[m] first (may be null); scratch holds the per-block
// partials until sums has added them up.
// (room also for the partial sums that softmax_xent and a product that makes C[M x N] leave)
size_t colsum_workspace_bytes(int64_t M, int32_t N);
grp_status launch_colsum_scaled(const float* A, int64_t M, int32_t N, int64_t lda, const float* rowmul,
                                float* out, void* scratch, StepSums& sums, hipStream_t st);
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
// a, b -> packed pairs hi, mid, lo with a = hi.x + mid.x + lo.x exactly.
__device__ __forceinline__ void split2(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{a, b}), bf16x2));
    const floatx2 r = {a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xFFFF0000u)};
    mid = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
    const float la = r.x - __uint_as_float(mid << 16), lb = r.y - __uint_as_float(mid & 0xFFFF0000u);
    lo = __builtin_amdgcn_perm(__float_as_uint(lb), __float_as_uint(la), 0x07060302u);
}
// An operand B of an NT product as its kernels read it: split into three bf16 planes (fp32 = hi + mid + lo, exactly), in tiles of 32 k.
// Tile kt, plane p and row n have 64 bytes at ((kt * 3 + p) * rows + n) * 64, in four places of eight k: place q ^ ((n >> 1) & 3) holds the k
// 4 q .. 4 q + 3 and 16 + 4 q .. 16 + 4 q + 3.  Rows and k that do not exist are zero, up to bt_plane_rows rows (what tiles of any
// width read) and whole tiles.
inline int32_t bt_plane_rows(int64_t n) { return (int32_t)std::max(round_up(n, 128), round_up(n, 96)); }
inline size_t bt_planes_bytes(int64_t k, int32_t rows) { return (size_t)cdiv(k, 32) * 3 * rows * 64; }
__host__ __device__ inline int64_t bt_planes_at(int k, int n, int plane, int rows) {      // the byte of element (n, k)
    const int kt = k >> 5, k32 = k & 31;
    return ((int64_t)(kt * 3 + plane) * rows + n) * 64 + 16 * (((k32 & 15) >> 2) ^ ((n >> 1) & 3)) + 2 * ((k32 & 3) + (k32 >> 4) * 4);
}
// Weight re-packing jobs of one step (at most four per layer), run by a single launch: a matrix of the parameters, or its transpose,
// times a scale, zero-padded, as fp32 and as planes.
struct PackJob {
    uint32_t in;             // element of the parameters
    uint32_t out, planes;    // units of 16 bytes of the workspace (planes 0: none)
    float scale;             // every element is multiplied by this
    uint16_t rows, cols;     // as written
    uint16_t out_rows;       // fp32 rows written (zeros from `rows` on)
    uint16_t ld4;            // their pitch in 16 bytes
    uint16_t row0, plane_rows;     // the planes' row of the first row; their rows in all
    uint16_t dom_rows;       // rows that this job writes to either
    uint16_t transpose;      // the matrix is stored as [cols x rows]
};
template <int MOST> struct PackJobsOf {
    const float* theta = nullptr;
    char* base = nullptr;    // the workspace
    int32_t n = 0;
    uint32_t begin[MOST + 1] = {0};      // pairs of elements
    PackJob job[MOST];
};
using PackJobs = PackJobsOf<4 * GRP_MAX_LAYERS>;
// Appends a job for the matrix in[rows x cols], or its transpose.  out: round_up(width, 4) columns and at least out_rows_pad rows.  planes
// (may be null): from row plane_row0 on, up to plane_rows if last, else as many rows as out has.
void pack_jobs_add(PackJobs& jobs, const float* in, int32_t rows, int32_t cols, bool transpose, int32_t out_rows_pad,
                   float* out, int64_t ld_out, unsigned char* planes, int32_t plane_row0, int32_t plane_rows, bool last, float scale = 1.f);

// Inverted dropout of a layer's output (rows = local nodes, F columns), in place:
//   keep(v, f) = (mix(key + (l2g[node(v)] * F + f + 1) * GAMMA) >> 40) >= thresh;  a' = keep ? a * scale : 0.
// Plain layer: H holds the activation.  Residual layer (act != null): act holds the activation and
// is overwritten with a'; H = a' + res.
struct DropoutPlan {
    bool on = false;
    uint32_t thresh = 0;
    float scale = 1.f;
    uint64_t seed = 0, batch_id = 0;
    const uint64_t* batch_id_dev = nullptr;   // when set: the batch id is read on the device instead
};
DropoutPlan dropout_plan(const grp_step_opts* o);
uint64_t dropout_layer_key(const DropoutPlan& d, int layer);
grp_status launch_dropout(const DropoutPlan& d, int layer, const int64_t* l2g, int64_t n, int32_t F, float* H, int64_t ldh,
                          float* act, int64_t ld_act, const float* res, int64_t ld_res, hipStream_t st,
                          const int32_t* node_of_row = nullptr /*row i is local node node_of_row[i] (null: i)*/,
                          const int64_t* n_dev = nullptr /*when set: the real row count (on the device), n an upper bound*/);
// Y[i, :F] = rowscale[i] * X[i, :F] (whole 16-byte column groups)
grp_status launch_scale_rows(const float* X, int64_t ldx, const float* rowscale, int64_t n, int32_t F, float* Y, int64_t ldy,
                             hipStream_t st, const int64_t* n_dev = nullptr /*as for launch_dropout*/);
// Y[i, :] = [X[i, :F] | 0 ...] up to the pitch ldy
grp_status launch_pad_rows(const float* X, int64_t ldx, int64_t n, int32_t F, float* Y, int64_t ldy, hipStream_t st);
// out[i] = in[i] * s
grp_status launch_scale_copy(const float* in, float s, float* out, int64_t n, hipStream_t st);

// Graph attention model (full-graph mode): workspace size and the whole train step.
size_t gat_step_workspace_bytes(const grp_partition_t* part, const grp_model_desc* m);
// Where layer `layer`'s stored output lives inside a workspace laid out for this partition and model.
void gat_step_activation(const grp_partition_t* part, const grp_model_desc* m, void* ws, size_t ws_bytes, int layer,
                         const float** out, int64_t* ld);
grp_status gat_step(const grp_partition_t* g, const grp_model_desc* m, const grp_step_opts* o, const void* X,
                    const int32_t* labels, const uint8_t* mask, const float* theta, void* ws, size_t ws_bytes,
                    hipStream_t st, float* grad, grp_step_stats* stats);

// Coverage statistics over the loss nodes and the weighted softmax cross-entropy.
size_t stats_workspace_bytes(int64_t n);
// nnz_used = nnz_const + the sum of the n_parts device counters nnz_parts[i][0]; or, when the device counter
// *bad_seeds is set and positive, minus that count (the record of a step whose seed list was invalid).
struct StatsIn {
    int64_t n_loss = 0;
    const int32_t* nodes = nullptr;                    // null: 0 .. n_loss - 1 by mask
    const uint8_t* mask = nullptr;
    const int32_t* d_local = nullptr;
    const int64_t* d_global = nullptr;
    const int32_t* sampled_count = nullptr;            // null: full graph
    int64_t nnz_const = 0;
    const int64_t* const* nnz_parts = nullptr;         // HOST array of device pointers
    int n_parts = 0;
    void* scratch = nullptr;                           // stats_workspace_bytes
    const double *w_local = nullptr, *w_global = nullptr;      // weight masses: full graph
    const int64_t* bad_seeds = nullptr;
};
// What a step does before its first layer, in one launch: the statistics' partial sums, the degree scales (inv_in = 1/max(d_in,1);
// r = 1/sqrt(max(d_in+sl,1)); s = 1/sqrt(max(d_out+sl,1)); rinv = 1/r; n = 0: none) and the re-packed weights (may be none).
struct DegreeScales {
    const int32_t *d_in = nullptr, *d_out = nullptr;
    int64_t n = 0;
    int sl = 0;
    float *inv_in = nullptr, *r = nullptr, *s = nullptr, *rinv = nullptr;      // each may be null
};
struct StepPrelude {
    StatsIn stats;
    DegreeScales degrees;
    PackJobs pack;
};
grp_status launch_prelude(const StepPrelude& pre, hipStream_t st);
// Reads the statistics' partial sums that launch_prelude left in in.scratch, writes the whole record.
grp_status launch_softmax_xent(const StatsIn& in, int32_t C, const float* Z, int64_t ldz,
                               const int32_t* labels, int32_t node_level,
                               const float* rowscale /*null; multiplies dZ rows*/,
                               float* dZ, int64_t lddz, grp_step_stats* stats, hipStream_t st,
                               StepSums* sums = nullptr /*when set: the record is left to it*/,
                               float* col_part = nullptr /*colsum_workspace_bytes; when set: and the column sums of dZ before rowscale*/,
                               float* col_out = nullptr);
constexpr int XENT_COLS_MOST = 192;       // classes up to which it makes them
// inv[v] = mass[v] > 0 ? 1 / mass[v] : 0
grp_status launch_inverse_mass(const double* mass, int64_t n, float* inv, hipStream_t st);

grp_status launch_fill_zero(void* p, size_t bytes, hipStream_t st);

}  // namespace grp

// ---------------------------------------------------------------- device primitives (partition.hip)
namespace grp {
// rocPRIM wrappers with caller-provided temporary storage (sizes from the *_temp_bytes calls).
size_t scan_temp_bytes(int64_t count);
grp_status exclusive_scan_i64(void* temp, size_t temp_bytes, const int64_t* in, int64_t* out, int64_t count,
                              hipStream_t st);
grp_status exclusive_scan_i32(void* temp, size_t temp_bytes, const int32_t* in, int32_t* out, int64_t count,
                              hipStream_t st);
// out[i] = number of set bits in words[0 .. i), i in [0, count): reads `count` words
grp_status exclusive_scan_popcount(void* temp, size_t temp_bytes, const uint32_t* words, int32_t* out, int64_t count,
                                   hipStream_t st);
// The split schedule of the long rows of a device pointer array, written into caller-provided device
// arrays without a host pass: out->n_long / n_chunks are set to the capacities (the launches cover
// them) and the slots beyond the real counts are filled so that they do nothing (row -1, empty
// chunks).  Capacities must cover every possible schedule: cap_long >= nnz / SPMM_LONG_ROW,
// cap_chunks >= nnz / SPMM_CHUNK + cap_long.  scanned: [n + 1] int64 scratch.
grp_status build_long_rows_device(const int64_t* ptr_dev, int64_t n, LongRows* out, int64_t cap_long, int64_t cap_chunks,
                                  int64_t* scanned, void* scan_tmp, size_t scan_bytes, hipStream_t st);

// ---- CSR and CSC from unordered keys (buckets.hip)
struct BucketPlan {
    int row_bits, id_bits;               // of a packed key: row within its bucket, other end
    int n_buckets;                       // of a direction
};
bool bucket_plan(int64_t n, int64_t nnz, BucketPlan* p);      // false: sizes that are not built this way
size_t bucket_scratch_bytes(const BucketPlan& p, int64_t nnz);
grp_status bucket_build(grp_partition_t* h, const BucketPlan& p, uint64_t* keys, uint64_t* packed, void* scratch, int64_t (&long_edges)[2],
                        bool* done, hipStream_t st, bool csc_alone = false);          // *done = false: refused, and the keys as they were (csc_alone: lost)

// M(x): the SplitMix64 finaliser of x + 0x9E3779B97F4A7C15 (the sampler's and the seed order's hash step)
__host__ __device__ __forceinline__ uint64_t mixM(uint64_t x) {
    uint64_t z = x + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// A helper stream beside a caller's stream, for work of a step that is off its critical path: the caller's
// stream records fork[i], the helper waits for it, works, records `join`, and the caller's stream waits for
// `join` before it needs the result (a fork and join that a graph capture of the caller's stream follows).
// Null when none can be had (creation failed, or the first request for this stream came while it was being
// captured): the work then stays on the caller's stream.  Calls that use the same caller stream from
// several host threads at once would mix up the events; the steps of one stream come from one thread.
struct SideLane {
    hipStream_t stream = nullptr;
    hipEvent_t fork[GRP_MAX_LAYERS] = {};
    hipEvent_t join = nullptr;
};
SideLane* side_lane(hipStream_t main);

// ---------------------------------------------------------------- blocks and sampling (sampler.hip)
// One bipartite message-passing layer.  Rows of `ptr/idx` are the layer's outputs
// (destinations); `idx` indexes rows of the layer's input matrix.  The outputs are the first
// n_dst inputs unless `self_rows` says where output i's own input row is stored.
struct Block {
    int64_t n_dst = 0, n_in = 0, nnz = 0;
    const int64_t* ptr = nullptr;
    const int32_t* idx = nullptr;
    const int64_t* ptrT = nullptr;       // transposed structure over the n_in inputs (null if unused)
    const int32_t* idxT = nullptr;
    const LongRows* long_fwd = nullptr;
    const LongRows* long_bwd = nullptr;
    const int32_t* self_rows = nullptr;  // [n_dst] or null (row i)
    float* inv_in = nullptr;             // [n_dst] 1 / max(row length, 1); weighted: 1 / local weight mass (0 if none)
    const int32_t* dst_nodes = nullptr;  // mini-batch: partition-local id of every destination row (null: row i is node i)
    const float* val = nullptr;          // weighted partitions: edge weights in ptr/idx order
    const float* valT = nullptr;         //                      and in ptrT/idxT order
    // Sampled blocks: n_dst, n_in and nnz above are upper bounds (from the seeds and fanouts) that size the
    // launches, and the real sizes live on the device (ptr and ptrT are valid up to the bounds: the rows
    // past the real ones are empty).  Null for a block whose sizes the host knows (n_in_dev is also null for
    // the input-side block, whose inputs are the partition's n nodes).
    const int64_t* n_dst_dev = nullptr;
    const int64_t* n_in_dev = nullptr;
};

struct SamplerBounds {                   // upper bounds per layer, from seeds and fanouts alone
    int64_t dst[GRP_MAX_LAYERS], nnz[GRP_MAX_LAYERS], src[GRP_MAX_LAYERS];
};
void sampler_bounds(int64_t n, int64_t n_seeds, const int32_t* fanouts, int k, SamplerBounds* out);
size_t sampler_workspace_bytes(int64_t n, const SamplerBounds& b, int k);
// Isolated k-hop sampling inside the partition; fills blocks[0..k) (layer 0 = input side).
// Layer 0's idx holds partition-local node ids (rows of the feature matrix) and its self_rows
// the destinations' ids; deeper layers are relabelled to block-local indices.  seeds_out
// receives the device pointer of the seed list; nnz_parts_dev[k] the per-layer edge counts
// (device); *bad_seeds_dev the number of seeds outside [0, n) (device; such a seed is replaced by node 0).
// Nothing here waits for the device: every launch is sized by the bounds and reads the real sizes from
// device memory, so the whole step can be queued (or captured in a graph) at once.
grp_status sample_blocks(const grp_partition_t* part, const grp_step_opts* opts, int k, void* ws, size_t ws_bytes,
                         Block* blocks, LongRows* long_bwd_store, const int64_t** nnz_parts_dev,
                         const int32_t** seed_counts_dev, const int64_t** bad_seeds_dev, hipStream_t st,
                         hipEvent_t* transposed_ready);
// *transposed_ready: null, or the event the caller's stream has to wait for before it reads a block's
// transposed structure (ptrT, idxT, long_bwd): those are built on a helper stream beside the sampling of the
// next layers, since only the backward pass reads them.
grp_status sampler_block_view(const grp_partition_t* part, const grp_step_opts* o, int k, void* ws, size_t ws_bytes, int layer,
                              grp_block_view_t* out);
}  // namespace grp

namespace grp {
// Bump allocator over a caller-provided workspace (null base: only measures).
struct Bump {
    char* base;
    size_t cap, off = 0;
    bool measure;
    Bump(void* b, size_t c) : base((char*)b), cap(c), measure(b == nullptr) {}
    template <typename T> T* take(size_t count) {
        off = (off + 255) & ~(size_t)255;
        T* p = measure ? nullptr : (T*)(base + off);
        off += count * sizeof(T);
        return p;
    }
    size_t total() const { return (off + 255) & ~(size_t)255; }
};
}  // namespace grp
