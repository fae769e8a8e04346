// Source-sliced schedule of the long rows of a CSR-like structure (built once with the partition).
//
// Why: a gather-bound aggregation over a graph without locality misses the L2 on almost every neighbour
// row (measured on a 2^24-node, 2^32-edge share: 0.82 line fills per edge), because the rows gathered
// at any one time are spread over all n sources.  The rows that hold most of the edges are long
// (96 % of the edges of a share with that mean degree sit in the fifth of the rows that are longer than 128 edges), and a row's sources are
// sorted, so a long row can be cut where its sources cross from one range of node ids into the next: the
// node ids are divided into SLICES = 64 equal ranges, every long row is cut at the boundaries between them
// (where the piece so far is long enough to be worth a task), and every piece into tasks of at most SLICE_TASK_MAX edges
// (a wavefront walks a task in passes of SLICE_PIECE edges).  The tasks are then processed slice by slice: at any one
// time the whole chip gathers from one 64th of the nodes, whose frequently used rows stay in the L2
// (measured with the sources restricted to one 64th: 0.14 fills per edge).  A task's result is a partial
// row; a long row's partial rows are added in task order (ascending source, the row's own edge order) by the
// combine pass, so the result does not depend on scheduling.
//
// Layout: tasks are numbered row-major (a long row's tasks are consecutive: row_task[j] .. row_task[j+1]),
// and the records are stored in processing order: by slice, and inside a slice in row order but for workgroups that ran side by side,
// so that neighbouring workgroups read neighbouring pieces of the index array.
#include "common.h"

#include <atomic>

#include <rocprim/rocprim.hpp>

namespace grp {

static_assert((SLICES & (SLICES - 1)) == 0, "the ranges are a power of two");
static std::atomic<int64_t> g_slice_min_nodes{(int64_t)1 << 19};
static std::atomic<int32_t> g_slice_min_percent{25};

static __device__ __forceinline__ int64_t lower_bound_idx(const int32_t* __restrict__ idx, int64_t b, int64_t e, int64_t want) {
    while (b < e) {
        const int64_t mid = (b + e) >> 1;
        if ((int64_t)idx[mid] < want) b = mid + 1; else e = mid;
    }
    return b;
}

// What the kernels below know of a direction (n_long = 0: no schedule is built for it).
struct SliceJob {
    const int64_t* ptr;
    const int32_t* idx;
    const int32_t* long_row;
    int64_t n_long;
    int64_t* row_task;               // [n_long + 1] tasks of every long row, then their prefix sum
    unsigned long long* slice_at;    // [SLICES] tasks of every slice, then where its next one goes
    SliceTask* tasks;
};
struct SliceJobs { SliceJob d[2]; };

// One wavefront per long row, sixteen rows per workgroup; blockIdx.y: the direction.  Lane s finds where the row's sources enter slice
// s; the row is then cut at such a
// boundary wherever the piece before it has reached SLICE_MIN_PIECE edges (a row of 600 edges is not worth 64
// pieces of 9: a piece costs a partial row and ~200 instructions; see the measurements beside the constant), and every piece into tasks of at most
// SLICE_TASK_MAX edges.  A task belongs to the slice of its first edge.  EMIT = false: the number of tasks of every row and slice.
// EMIT = true: the task records (row-major numbering from row_task[j]) to their slices: a workgroup reserves one run of places
// per slice, so that inside a slice the records keep the rows' order but for the workgroups in flight.
constexpr int SLICE_ROWS = 16;
template <bool EMIT>
__global__ __launch_bounds__(64 * SLICE_ROWS) void slice_rows_kernel(SliceJobs jobs, int shift, int min_piece) {
    __shared__ int64_t cut_s[SLICE_ROWS][SLICES + 1];
    __shared__ uint32_t in_slice[SLICES];
    __shared__ unsigned long long run[SLICES];
    const SliceJob& job = jobs.d[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((int64_t)blockIdx.x * SLICE_ROWS >= job.n_long) return;
    const int64_t j = (int64_t)blockIdx.x * SLICE_ROWS + wave;
    const int64_t r = j < job.n_long ? job.long_row[j] : -1;   // (-1 is also an unused slot of a schedule built to its capacity)
    const int64_t b = r >= 0 ? job.ptr[r] : 0, e = r >= 0 ? job.ptr[r + 1] : 0;
    for (int sl = threadIdx.x; sl < SLICES; sl += 64 * SLICE_ROWS) in_slice[sl] = 0u;
    if (r >= 0)
        for (int sl = lane; sl < SLICES; sl += 64) cut_s[wave][sl] = sl == 0 ? b : lower_bound_idx(job.idx, b, e, (int64_t)sl << shift);
    if (lane == 0) cut_s[wave][SLICES] = e;
    __syncthreads();
    auto walk = [&](auto piece) {                              // piece(from, to, slice, tasks): the same in every lane
        int64_t from = b;                                      // start of the current piece
        int from_slice = 0;
        for (int s = 1; s <= SLICES && r >= 0; ++s) {
            const int64_t at = cut_s[wave][s];
            const bool close = s == SLICES || at - from >= min_piece;
            if (!close) continue;
            piece(from, at, from_slice, (at - from + SLICE_TASK_MAX - 1) / SLICE_TASK_MAX);
            from = at;
            from_slice = s;
        }
    };
    int64_t count = 0;
    walk([&](int64_t, int64_t, int slice, int64_t nt) {
        if (lane == 0 && nt > 0) atomicAdd(&in_slice[slice], (uint32_t)nt);
        count += nt;
    });
    if (!EMIT && lane == 0 && j < job.n_long) job.row_task[j] = count;
    __syncthreads();
    for (int sl = threadIdx.x; sl < SLICES; sl += 64 * SLICE_ROWS)
        if (in_slice[sl]) {
            run[sl] = atomicAdd(&job.slice_at[sl], (unsigned long long)in_slice[sl]);
            in_slice[sl] = 0u;
        }
    if (!EMIT) return;
    __syncthreads();
    int64_t t = r >= 0 ? job.row_task[j] : 0;
    walk([&](int64_t from, int64_t to, int slice, int64_t nt) {
        if (nt <= 0) return;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&in_slice[slice], (uint32_t)nt);
        at = __shfl(at, 0, 64);
        for (int64_t i = lane; i < nt; i += 64) {
            SliceTask rec;
            rec.begin = from + i * SLICE_TASK_MAX;
            rec.id = (uint32_t)(t + i);
            rec.len = (uint32_t)(to - rec.begin < SLICE_TASK_MAX ? to - rec.begin : SLICE_TASK_MAX);
            job.tasks[run[slice] + at + i] = rec;
        }
        t += nt;
    });
}

// The prefix sums of row_task (rows: not done elsewhere) and slice_at, a workgroup per direction.
__global__ __launch_bounds__(1024) void slice_scan_kernel(SliceJobs jobs, int rows) {
    __shared__ int64_t wave_sum[16];
    const SliceJob& job = jobs.d[blockIdx.x];
    if (job.n_long == 0) return;
    constexpr int PER = 8;
    int64_t base = 0, total;
    for (int64_t j0 = 0; rows && j0 < job.n_long; j0 += 1024 * PER) {
        int64_t v[PER], sum = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t j = j0 + PER * (int)threadIdx.x + i;
            v[i] = j < job.n_long ? job.row_task[j] : 0;
            sum += v[i];
        }
        int64_t at = base + block_scan<16>(sum, wave_sum, total);
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int64_t j = j0 + PER * (int)threadIdx.x + i;
            if (j < job.n_long) job.row_task[j] = at;
            at += v[i];
        }
        base += total;
    }
    if (rows && threadIdx.x == 0) job.row_task[job.n_long] = base;
    static_assert(SLICES <= 1024, "a thread per slice");
    const int64_t mine = threadIdx.x < SLICES ? (int64_t)job.slice_at[threadIdx.x] : 0;
    const int64_t at = block_scan<16>(mine, wave_sum, total);
    if (threadIdx.x < SLICES) job.slice_at[threadIdx.x] = (unsigned long long)at;
}

// *total += the edges of the listed rows (one atomic per wavefront)
__global__ __launch_bounds__(256) void long_edges_kernel(const int64_t* __restrict__ ptr, const int32_t* __restrict__ long_row,
                                                         int64_t n_long, unsigned long long* __restrict__ total) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int64_t len = 0;
    if (j < n_long) {
        const int64_t r = long_row[j];
        if (r >= 0) len = ptr[r + 1] - ptr[r];
    }
    for (int o = 32; o > 0; o >>= 1) len += __shfl_down(len, o, 64);
    if ((threadIdx.x & 63) == 0 && len > 0) atomicAdd(total, (unsigned long long)len);
}

// Builds tasks / row_task for the long rows listed in the handle (allocations owned by the handle).  Leaves a direction without them
// (n_tasks = 0) when the structure is too small to gain.  long_edges: the edges of each direction's long rows (negative: counted here).
grp_status build_slice_tasks(grp_partition_t* h, const int64_t (&long_edges)[2], hipStream_t st) {
    const int64_t n = h->n, nnz = h->nnz;
    LongRows* const lr[2] = {&h->csr_long, &h->csc_long};
    for (LongRows* l : lr) { l->n_tasks = 0; l->tasks = nullptr; l->row_task = nullptr; }
    if (n < g_slice_min_nodes.load() || (lr[0]->n_long <= 0 && lr[1]->n_long <= 0)) return GRP_OK;
    int shift = 0;
    while (((n - 1) >> shift) >= SLICES) ++shift;
    SliceJobs jobs{{{h->rowptr, h->col, lr[0]->long_row, lr[0]->n_long, nullptr, nullptr, nullptr},
                    {h->colptr, h->row, lr[1]->long_row, lr[1]->n_long, nullptr, nullptr, nullptr}}};
    struct Temp {                          // freed on return
        void* p = nullptr;
        ~Temp() { pool_free(p); }
    } slice_at, scan_tmp;
    constexpr size_t AT = SLICES + 1;      // (the last: edges)
    if (pool_alloc(&slice_at.p, 2 * AT * sizeof(unsigned long long)) != hipSuccess) {
        (void)hipGetLastError();
        return fail(GRP_ENOMEM, "slice schedule: counters");
    }
    unsigned long long* const at = (unsigned long long*)slice_at.p;
    GRP_TRY(launch_fill_zero(at, 2 * AT * sizeof(unsigned long long), st));
    int64_t edges[2] = {long_edges[0], long_edges[1]};
    if (edges[0] < 0 || edges[1] < 0) {
        unsigned long long counted[2 * AT];
        for (int d = 0; d < 2; ++d)
            if (jobs.d[d].n_long > 0)
                hipLaunchKernelGGL(long_edges_kernel, dim3((unsigned)cdiv(jobs.d[d].n_long, 256)), dim3(256), 0, st, jobs.d[d].ptr, jobs.d[d].long_row,
                                   jobs.d[d].n_long, at + d * AT + SLICES);
        GRP_LAUNCH_CHECK();
        GRP_HIP(hipMemcpyAsync(counted, at, sizeof counted, hipMemcpyDeviceToHost, st));
        GRP_HIP(hipStreamSynchronize(st));
        for (int d = 0; d < 2; ++d) edges[d] = (int64_t)counted[d * AT + SLICES];
    }
    auto give_up = [&](grp_status s) {
        for (SliceJob& j : jobs.d) { pool_free(j.tasks); pool_free(j.row_task); }
        return s;
    };
    int64_t most = 0;
    for (int d = 0; d < 2; ++d) {          // the long rows' share of the edges decides whether the schedule pays
        SliceJob& j = jobs.d[d];
        if (j.n_long <= 0 || edges[d] * 100 < nnz * (int64_t)g_slice_min_percent.load()) { j.n_long = 0; continue; }
        // A row's pieces but its last have SLICE_MIN_PIECE edges, a piece's tasks but its last SLICE_TASK_MAX: that many tasks at most (on
        // graphs with hubs nine tenths of it are used; waiting for the exact number would cost more than it saves).
        const int64_t cap = edges[d] / SLICE_MIN_PIECE + edges[d] / SLICE_TASK_MAX + j.n_long;
        if (cap >= ((int64_t)1 << 32)) { j.n_long = 0; continue; }       // more tasks than a 32-bit id holds
        j.slice_at = at + d * AT;
        if (pool_alloc((void**)&j.row_task, (size_t)(j.n_long + 1) * sizeof(int64_t)) != hipSuccess ||
            pool_alloc((void**)&j.tasks, (size_t)cap * sizeof(SliceTask)) != hipSuccess) {
            (void)hipGetLastError();
            return give_up(fail(GRP_ENOMEM, "slice schedule: %lld task records", (long long)cap));
        }
        if (j.n_long > most) most = j.n_long;
    }
    if (most == 0) return GRP_OK;
    const dim3 grid((unsigned)cdiv(most, SLICE_ROWS), 2);
    hipLaunchKernelGGL(slice_rows_kernel<false>, grid, dim3(64 * SLICE_ROWS), 0, st, jobs, shift, SLICE_MIN_PIECE);
    // one workgroup takes 8192 rows a round (about 3 us); the library's scan takes two launches per direction
    const bool many = most > ((int64_t)1 << 16);
    if (many) {
        size_t need = 0;
        auto scan = [&](const SliceJob& j) {
            return rocprim::exclusive_scan(scan_tmp.p, need, j.row_task, j.row_task, (int64_t)0, (size_t)(j.n_long + 1), rocprim::plus<int64_t>(), st);
        };
        const SliceJob& big = jobs.d[0].n_long >= jobs.d[1].n_long ? jobs.d[0] : jobs.d[1];
        bool ok = scan(big) == hipSuccess && pool_alloc(&scan_tmp.p, need ? need : 4) == hipSuccess;
        for (const SliceJob& j : jobs.d)
            if (ok && j.n_long > 0) ok = launch_fill_zero(j.row_task + j.n_long, sizeof(int64_t), st) == GRP_OK && scan(j) == hipSuccess;
        if (!ok) {
            (void)hipGetLastError();
            return give_up(fail(GRP_EHIP, "slice schedule: scan failed"));
        }
    }
    hipLaunchKernelGGL(slice_scan_kernel, dim3(2), dim3(1024), 0, st, jobs, many ? 0 : 1);
    hipLaunchKernelGGL(slice_rows_kernel<true>, grid, dim3(64 * SLICE_ROWS), 0, st, jobs, shift, SLICE_MIN_PIECE);
    int64_t n_tasks[2] = {0, 0};
    hipError_t e = hipGetLastError();
    for (int d = 0; d < 2 && e == hipSuccess; ++d)
        if (jobs.d[d].n_long > 0)
            e = hipMemcpyAsync(&n_tasks[d], jobs.d[d].row_task + jobs.d[d].n_long, sizeof(int64_t), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return give_up(fail(GRP_EHIP, "slice schedule: %s", hipGetErrorString(e)));
    for (int d = 0; d < 2; ++d) {
        if (jobs.d[d].n_long == 0) continue;
        lr[d]->n_tasks = n_tasks[d];
        lr[d]->tasks = jobs.d[d].tasks;
        lr[d]->row_task = jobs.d[d].row_task;
    }
    return GRP_OK;
}

}  // namespace grp

extern "C" grp_status grp_set_slice_policy(int64_t min_nodes, int32_t min_long_edge_percent) {
    if (min_nodes < 1 || min_long_edge_percent < 0 || min_long_edge_percent > 100)
        return grp::fail(GRP_EINVAL, "grp_set_slice_policy: %lld nodes, %d %%", (long long)min_nodes, min_long_edge_percent);
    grp::g_slice_min_nodes.store(min_nodes);
    grp::g_slice_min_percent.store(min_long_edge_percent);
    return GRP_OK;
}
