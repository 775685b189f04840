// The plan built on the device from per-row kept counts (section 3.2): each row's
// block size from its density, the rows grouped by block size (ascending; original
// order inside a group) and each row's first slot -- the same plan darb_plan_create_counts
// builds on the host, written straight into the plan workspace.
//
// Rounding in integers.  With d = count / N, f = the largest power of two with
// f * count <= N (the largest with f * d <= 1): d is itself a power-of-two fraction when
// f * count == N, and then both directions give b = f; otherwise rounding the density
// up gives b = f and rounding it down b = 2f.  Floor mode always rounds up; paper mode
// rounds up when d >= D, i.e. count * M >= kept (D = kept / (M N)).  A row with count 0
// gets b_max; b is clamped to [b_min, b_max].  These are the host rule's results: the
// host compares fp64 quotients, and two distinct quotients of this size never round
// to the same double.
//
// Up to kPlanOneRows rows, one launch of one workgroup, which holds every row's block
// size in registers; it hands the group summary to the host itself, through pinned memory
// and a flag, so that the host neither copies nor waits for the stream.  The rows of such
// a plan are few enough that three launches, a copy and the wait for it cost several times
// the work: 4096 rows, 5.0 + 2.6 + 3.4 us of kernels and 2.3 us of copy before, 8.3 us
// now, and a compression of 4096 x 9216 fp32 (pruning, plan, encode, packing, codes) 158
// -> 112 us, part of it from the pruning.  (Every thread fencing for itself: 12.4 us.)  The
// whole call, host and all: 22.6 us at 4096 rows, 28.7 at 8192, 36.4 with three launches, and
// 39 to 41 with 16 rows per thread at 10240 to 16384 rows.
//
// Otherwise three launches: per-row block size and per-workgroup group counts; one workgroup scans
// those counts into group starts and each workgroup's first position per group (and
// writes the group summary the host reads back); each row then takes its place --
// workgroup start plus its rank among the workgroup's rows of the same group, counted
// with ballots -- which gives the storage order, the first slot and the per-row table.
#include "darb_internal.h"

namespace darb {
namespace {

constexpr int kPlanThreads = 1024;
constexpr int kPlanWaves = kPlanThreads / kWave;
constexpr int kGroups = kMaxBins;               // log2 b = 0 .. 7
constexpr int64_t kPlanOneRows = 8 * kPlanThreads;

__device__ __forceinline__ int row_log2b_counts(int64_t c, int64_t N, int64_t M, int64_t kept,
                                                int mode, int lmin, int lmax) {
    if (c <= 0) return lmax;
    if (c > N) c = N;
    int l = 0;                                  // largest l with (c << l) <= N, or past lmax
#pragma unroll
    for (int i = 1; i <= kMaxLog2B + 1; ++i) l += (c << i) <= N ? 1 : 0;
    const bool exact = (c << l) == N;
    const bool up = (mode == DARB_ROUND_FLOOR) || (c * M >= kept);
    if (!up && !exact) ++l;
    return l < lmin ? lmin : (l > lmax ? lmax : l);
}

// The LSTM sequence launch needs to know, before it is chosen, the most chunks that one of
// its workgroups would hold.  The wave's rows (one per active lane, block size 2^l) add
// theirs to their members' in `held` (LDS, zeroed): consecutive rows have few members, so
// a member at a time and one atomic each...
__device__ __forceinline__ void lstm_hold(int (&held)[kLstmMembers], int64_t N, int64_t r, int l,
                                          bool active) {
    const int member = int(uint32_t(r) % uint32_t(N) / uint32_t(lstm_units(N)));
    for (uint64_t left = __ballot(active); left != 0;) {     // wave-uniform
        const int m = __builtin_amdgcn_readlane(member, __ffsll((unsigned long long)left) - 1);
        const uint64_t same = __ballot(active && member == m);
        int sum = 0;
#pragma unroll
        for (int v = 0; v < kGroups; ++v)
            sum += __popcll(__ballot(l == v) & same) * int(lstm_row_chunks(N, v));
        if ((threadIdx.x & (kWave - 1)) == 0) atomicAdd(&held[m], sum);
        left &= ~same;
    }
}
// ... and the largest of them, for every lane of the calling wave.
__device__ __forceinline__ int64_t lstm_most(const int (&held)[kLstmMembers]) {
    int v = held[threadIdx.x & (kLstmMembers - 1)];
#pragma unroll
    for (int m = kLstmMembers / 2; m >= 1; m >>= 1) {
        const int o = __shfl_xor(v, m, kWave);
        v = o > v ? o : v;
    }
    return v;
}

// Rank of this lane among the wave's active lanes below it with the same key, and
// the wave's count per key (every lane of the wave gets the same counts).
__device__ __forceinline__ int wave_rank(int key, bool active, int (&count)[kGroups]) {
    const uint64_t below = (uint64_t(1) << (threadIdx.x & (kWave - 1))) - 1;
    int rank = 0;
#pragma unroll
    for (int v = 0; v < kGroups; ++v) {
        const uint64_t m = __ballot(active && key == v);
        count[v] = __popcll(m);
        if (key == v) rank = __popcll(m & below);
    }
    return rank;
}

// Block sizes (into rowinfo's low byte) and each workgroup's row count per group.
__global__ __launch_bounds__(kPlanThreads) void plan_sizes_kernel(
    int64_t M, int64_t N, const int64_t *__restrict__ counts, int64_t kept, int mode, int lmin,
    int lmax, int64_t *__restrict__ rowinfo, int32_t *__restrict__ wg_counts) {
    __shared__ int part[kPlanWaves][kGroups];
    const int64_t r = int64_t(blockIdx.x) * kPlanThreads + threadIdx.x;
    const bool active = r < M;
    int l = 0;
    if (active) {
        l = row_log2b_counts(counts[r], N, M, kept, mode, lmin, lmax);
        rowinfo[r] = l;
    }
    int cnt[kGroups];
    wave_rank(l, active, cnt);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0)
        for (int v = 0; v < kGroups; ++v) part[wave][v] = cnt[v];
    __syncthreads();
    if (threadIdx.x < kGroups) {
        int s = 0;
        for (int w = 0; w < kPlanWaves; ++w) s += part[w][threadIdx.x];
        wg_counts[int64_t(blockIdx.x) * kGroups + threadIdx.x] = s;
    }
}

// One workgroup: group sizes and starts, and each workgroup's first position in each
// group (overwriting wg_counts).  summary: rows, first_row, first_elem, first_word,
// 8 int64 each, and the LSTM chunks.
__global__ __launch_bounds__(kPlanThreads) void plan_scan_kernel(
    int64_t M, int64_t N, int64_t nwg, const int64_t *__restrict__ rowinfo,
    int32_t *__restrict__ wg_counts, int64_t *__restrict__ summary) {
    __shared__ int64_t total[kGroups];
    __shared__ int64_t start[kGroups];
    __shared__ int held[kLstmMembers];
    const int v = threadIdx.x / kWave;                   // one wave per group
    const int lane = threadIdx.x & (kWave - 1);
    if (threadIdx.x < kLstmMembers) held[threadIdx.x] = 0;
    __syncthreads();
    if (lstm_shape(M, N))                                // uniform; few rows
        for (int64_t r0 = 0; r0 < M; r0 += kPlanThreads) {
            const int64_t r = r0 + threadIdx.x;
            lstm_hold(held, N, r, int(rowinfo[r < M ? r : M - 1] & 0xFF), r < M);
        }
    if (v < kGroups) {
        // rows of group v, summed in chunks of 64 workgroups
        int64_t s = 0;
        for (int64_t b = lane; b < nwg; b += kWave) s += wg_counts[b * kGroups + v];
        for (int m = kWave / 2; m >= 1; m >>= 1) s += __shfl_xor(s, m, kWave);
        if (lane == 0) total[v] = s;
    }
    __syncthreads();
    if (v == kGroups) {
        const int64_t most = lstm_most(held);
        if (lane == 0) summary[kSummaryLstm] = most;
    }
    if (threadIdx.x == 0) {
        int64_t row = 0, elem = 0, word = 0;
        for (int g = 0; g < kGroups; ++g) {
            const int64_t nblk = (N + (int64_t(1) << g) - 1) >> g;
            start[g] = row;
            summary[g] = total[g];
            summary[kGroups + g] = row;
            summary[2 * kGroups + g] = elem;
            if (g > 0) summary[3 * kGroups + g] = word;
            row += total[g];
            elem += total[g] * nblk;
            word += (total[g] * nblk + 31) / 32 * g;
        }
    }
    __syncthreads();
    if (v < kGroups) {
        // exclusive scan of group v's per-workgroup counts, 64 workgroups at a time
        int64_t base = start[v];
        for (int64_t b0 = 0; b0 < nwg; b0 += kWave) {
            const int64_t b = b0 + lane;
            const int64_t c = b < nwg ? wg_counts[b * kGroups + v] : 0;
            int64_t incl = c;
            for (int m = 1; m < kWave; m <<= 1) {
                const int64_t t = __shfl_up(incl, m, kWave);
                if (lane >= m) incl += t;
            }
            if (b < nwg) wg_counts[b * kGroups + v] = int32_t(base + incl - c);
            base += __shfl(incl, kWave - 1, kWave);
        }
    }
}

// Everything above and below in one workgroup: rows t * 1024 + thread, TILES of them per
// thread.  `host` (pinned): the summary, then the flag.  The tables are written back
// before the flag goes out: whoever the host tells about it finds them complete.
template <int TILES>
__global__ __launch_bounds__(kPlanThreads) void plan_one_kernel(
    int64_t M, int64_t N, const int64_t *__restrict__ counts, int64_t kept, int mode, int lmin,
    int lmax, int64_t *__restrict__ rowinfo, int32_t *__restrict__ perm, PlanSummary *host) {
    constexpr int kParts = TILES * kPlanWaves;           // (tile, wave) pairs, in row order
    constexpr int kPer = (kParts + kWave - 1) / kWave;   // of them per lane of the scan
    __shared__ int part[kGroups][kParts];                // rows of each pair, then the rows before
    __shared__ int64_t total[kGroups], first_row[kGroups], first_elem[kGroups];
    __shared__ int held[kLstmMembers];
    const int lane = int(threadIdx.x) & (kWave - 1);
    const int wave = int(threadIdx.x) / kWave;
    const bool lstm = lstm_shape(M, N);                  // uniform
    int64_t c[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {                    // all loads first
        const int64_t r = int64_t(t) * kPlanThreads + threadIdx.x;
        c[t] = counts[r < M ? r : M - 1];
    }
    if (lstm) {
        if (threadIdx.x < kLstmMembers) held[threadIdx.x] = 0;
        __syncthreads();
    }
    int l[TILES], rank[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int64_t r = int64_t(t) * kPlanThreads + threadIdx.x;
        l[t] = row_log2b_counts(c[t], N, M, kept, mode, lmin, lmax);
        int cnt[kGroups];
        rank[t] = wave_rank(l[t], r < M, cnt);
        if (lane == 0) {
#pragma unroll
            for (int v = 0; v < kGroups; ++v) part[v][t * kPlanWaves + wave] = cnt[v];
        }
        if (lstm) lstm_hold(held, N, r, l[t], r < M);
    }
    __syncthreads();
    if (wave < kGroups) {                                // one wave per group
        int own[kPer], sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int at = lane * kPer + i;
            own[i] = at < kParts ? part[wave][at] : 0;
            sum += own[i];
        }
        int incl = sum;
#pragma unroll
        for (int m = 1; m < kWave; m <<= 1) {
            const int o = __shfl_up(incl, m, kWave);
            if (lane >= m) incl += o;
        }
        int before = incl - sum;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int at = lane * kPer + i;
            if (at < kParts) part[wave][at] = before;
            before += own[i];
        }
        if (lane == kWave - 1) total[wave] = incl;
    }
    __shared__ int64_t most;
    if (wave == kGroups) most = lstm ? lstm_most(held) : 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t row = 0, elem = 0, word = 0;
        host->v[kSummaryLstm] = most;
        for (int g = 0; g < kGroups; ++g) {
            const int64_t nblk = (N + (int64_t(1) << g) - 1) >> g;
            first_row[g] = row;
            first_elem[g] = elem;
            host->v[g] = total[g];
            host->v[kGroups + g] = row;
            host->v[2 * kGroups + g] = elem;
            if (g > 0) host->v[3 * kGroups + g] = word;
            row += total[g];
            elem += total[g] * nblk;
            word += (total[g] * nblk + 31) / 32 * g;
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        const int64_t r = int64_t(t) * kPlanThreads + threadIdx.x;
        if (r < M) {
            const int in_group = part[l[t]][t * kPlanWaves + wave] + rank[t];
            const int64_t nblk = (N + (int64_t(1) << l[t]) - 1) >> l[t];
            perm[first_row[l[t]] + in_group] = int32_t(r);
            rowinfo[r] = ((first_elem[l[t]] + in_group * nblk) << 8) | l[t];
        }
    }
    // the barrier orders every wave's table stores before the flag's store, whose release at
    // system scope is cumulative: it makes them visible too (the barrier itself waits for
    // no other wave's stores)
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&host->ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Each row's storage position: its workgroup's first position in its group plus its
// rank among the workgroup's earlier rows of that group.
__global__ __launch_bounds__(kPlanThreads) void plan_place_kernel(
    int64_t M, int64_t N, const int32_t *__restrict__ wg_start,
    const int64_t *__restrict__ summary, int64_t *__restrict__ rowinfo,
    int32_t *__restrict__ perm) {
    __shared__ int part[kPlanWaves][kGroups];
    const int64_t r = int64_t(blockIdx.x) * kPlanThreads + threadIdx.x;
    const bool active = r < M;
    const int l = active ? int(rowinfo[r] & 0xFF) : 0;
    int cnt[kGroups];
    const int rank = wave_rank(l, active, cnt);
    const int wave = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0)
        for (int v = 0; v < kGroups; ++v) part[wave][v] = cnt[v];
    __syncthreads();
    if (!active) return;
    int before = 0;                                      // earlier waves' rows of group l
    for (int w = 0; w < wave; ++w) before += part[w][l];
    const int64_t pos = int64_t(wg_start[int64_t(blockIdx.x) * kGroups + l]) + before + rank;
    const int64_t nblk = (N + (int64_t(1) << l) - 1) >> l;
    const int64_t slot = summary[2 * kGroups + l] + (pos - summary[kGroups + l]) * nblk;
    perm[pos] = int32_t(r);
    rowinfo[r] = (slot << 8) | l;
}

}  // namespace

int64_t plan_device_scratch_bytes(int64_t M) {
    const int64_t nwg = (M + kPlanThreads - 1) / kPlanThreads;
    return 4 * kGroups * int64_t(sizeof(int64_t)) + nwg * kGroups * int64_t(sizeof(int32_t));
}

bool plan_one_launch(int64_t M) { return M <= kPlanOneRows; }

hipError_t launch_plan_one(int64_t M, int64_t N, const int64_t *counts, int64_t kept, int mode,
                           int lmin, int lmax, int32_t *perm, int64_t *rowinfo, PlanSummary *host,
                           hipStream_t s) {
#define DARB_PLAN_ONE(T)                                                                      \
    hipLaunchKernelGGL((plan_one_kernel<T>), dim3(1), dim3(kPlanThreads), 0, s, M, N, counts,  \
                       kept, mode, lmin, lmax, rowinfo, perm, host)
    if (M <= 4 * kPlanThreads) DARB_PLAN_ONE(4);
    else DARB_PLAN_ONE(8);
#undef DARB_PLAN_ONE
    return hipGetLastError();
}

hipError_t launch_plan_device(int64_t M, int64_t N, const int64_t *counts, int64_t kept, int mode,
                              int lmin, int lmax, int32_t *perm, int64_t *rowinfo, void *scratch,
                              hipStream_t s) {
    const int64_t nwg = (M + kPlanThreads - 1) / kPlanThreads;
    if (nwg > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
    int64_t *summary = static_cast<int64_t *>(scratch);
    int32_t *wg_counts = reinterpret_cast<int32_t *>(summary + 4 * kGroups);
    hipLaunchKernelGGL(plan_sizes_kernel, dim3(unsigned(nwg)), dim3(kPlanThreads), 0, s, M, N,
                       counts, kept, mode, lmin, lmax, rowinfo, wg_counts);
    hipLaunchKernelGGL(plan_scan_kernel, dim3(1), dim3(kPlanThreads), 0, s, M, N, nwg, rowinfo,
                       wg_counts, summary);
    hipLaunchKernelGGL(plan_place_kernel, dim3(unsigned(nwg)), dim3(kPlanThreads), 0, s, M, N,
                       wg_counts, summary, rowinfo, perm);
    return hipGetLastError();
}

}  // namespace darb
