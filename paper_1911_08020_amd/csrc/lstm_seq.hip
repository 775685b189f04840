// The recurrent part of the LSTM layer (section 4.1) as one launch over all time steps.
//
// One launch per step spends most of its time outside the product: the launch itself,
// then three dependent memory round trips (the unit's row table, its weights, the
// gathers of h).  Here workgroups stay resident for the whole sequence: each keeps the
// retained weights of its hidden units in registers and only h crosses workgroups.
//
// Split.  The batch is cut into groups of CPG columns; a recurrence only couples units of
// the same column, so groups never talk to each other.  Workgroup i belongs to group
// i % 8 and the hardware hands workgroup i to XCD i % 8, so a group's members share one
// XCD's L2, which is what makes the exchange of h cheap.  Members compare the numbers of
// the XCDs they run on before they rely on it.  A group's members split the hidden units
// evenly.
//
// Exchange.  h_t goes through a ring of three slots in the workspace.  A slot starts out
// filled with a sentinel (a NaN pattern that no stored h has) and a reader polls the data
// itself until no word is the sentinel: one memory round trip per step, no separate flag.
// Every word is read with a device-scope load.  It is written with a device-scope store
// unless the whole group runs on one XCD: then with a plain one (workgroup scope), for
// which the memory model promises other workgroups nothing.  What makes it right is the
// hardware: the vector caches write through, so an acknowledged store is in the XCD's one
// L2, and that is where the readers' loads go on the same XCD; equal XCC_ID registers are
// therefore a condition of correctness.  The test forces the other form too and asks for
// the same bits.  Having read all of h_{t-1},
// a member knows that every other member has finished with h_{t-2} (it published h_{t-1}
// after that), so it puts the sentinel back into its own part of that slot, waits until
// this is acknowledged, and only then publishes h_t: whoever sees h_t and later polls the
// slot for h_{t+1} cannot see the old h_{t-2}.
//
// Waiting is bounded.  All members must be on the chip at once: the grid is at most one
// workgroup per CU, and sequences take turns on a device, whatever their streams.  The
// turn is taken on the device, by the launch before the sequence, which then has all that
// its stream ordered before it behind it: who holds the turn waits for nobody else, so a
// sequence never waits for work that another stream has only queued.  (Ordered by the host
// with events, a layer waited for one queued earlier on another stream and with it for
// whatever that stream waited for, which could be this layer's own results.)  Other
// kernels hold CUs only until they end; another process could hold them for longer.  A
// member that has polled max_polls times for one step sets
// the failure flag and leaves, the others follow, and the last launch
// (lstm_finish_kernel) then computes the sequence again from the untouched initial
// state, one workgroup per batch column, which needs nobody else.  It sums in the same
// order, so the results are the same bits.
//
// H = 1024, T = 200, batch 32, fp16, 4.2 % kept: 2.9 us per step, against 7.3 us with a
// launch per step; a layer with its input products 1660 -> 741 us.  A step spends 0.8 us
// until the last member's h arrives, 0.3 us to put it into LDS and meet, 1.1 us on the
// gathers (LDS bank conflicts are about half of it), 0.4 us on the rows' sums and 0.3 us
// on the cell and the stores.
#include <hip/hip_fp16.h>

#include <mutex>

#include "darb_internal.h"
#include "lstm_cell.h"

namespace darb {
namespace {

constexpr int kSeqThreads = 512;
constexpr int kSeqXcds = 8;           // workgroups are handed to the XCDs in turn
constexpr int kSeqMembers = kLstmMembers;   // most workgroups per group: an XCD's CUs
constexpr int kSeqChunk = kLstmChunk;       // weights per chunk: one thread's unit of work
// chunks per thread, kept in registers (the LDS holds one sum of each)
constexpr int seq_resident(int cpg) { return cpg == 8 ? 2 : 3; }
constexpr int kSeqMaxRows = kSeqThreads;   // gate rows of a member: one thread each
constexpr int kSeqMaxNblk = 512;      // retained weights per row (at most 64 chunks)
constexpr uint32_t kSentinel = 0x7FDA5EEDu;   // a quiet NaN
constexpr int64_t kSeqMaxLds = 128 * 1024;
// reads of the turn, about 2 us each, before a sequence runs without it
constexpr uint32_t kTurnPolls = 1u << 22;
constexpr int kFinishThreads = 1024;
constexpr int kXccId = 20 | (31 << 11);       // s_getreg: all of the XCC_ID register

struct SeqArgs {
    const void *values;
    const uint8_t *offsets;
    const int64_t *rowinfo;
    const float *U;          // [4H x ldu]: input products, column t * batch + n
    const float *h0, *c0;    // [H x batch]
    float *h_seq;            // [H x ldu]
    float *h_out, *c_out;    // [H x batch]: written by the last launch only
    uint32_t *ring;          // [3][groups][H][CPG]
    uint32_t *failed;        // [0]: a member gave up; [1]: the sequence holds the turn
    int64_t ldu;
    int32_t H, T, batch, groups, members, units;   // units per member
    uint32_t max_polls;
    uint32_t far;            // device-scope stores wherever the members run
};

__device__ __forceinline__ int wave_uniform_i(int v) { return __builtin_amdgcn_readfirstlane(v); }

// One chunk in registers: the weights, and the LDS byte address of each one's column of
// h (below 2^16).  Slots past the row's end hold weight 0 and the address of a row of
// zeros, so they add +0.0 whatever h holds.  opaque() hides that the packed words are the
// same at every step: unpacked once for all steps they would take twice the registers.
template <typename Tw> struct Chunk;
template <> struct Chunk<float> {
    float w[kSeqChunk];
    uint32_t a[kSeqChunk / 2];
    __device__ __forceinline__ void set(int i, float v, uint32_t addr) {
        w[i] = v;
        if (i & 1) a[i / 2] |= addr << 16;
        else a[i / 2] = addr;
    }
    __device__ __forceinline__ float weight(int i) const { return w[i]; }
    __device__ __forceinline__ uint32_t addr(int i) const {
        return (i & 1) ? a[i / 2] >> 16 : a[i / 2] & 0xFFFFu;
    }
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int i = 0; i < kSeqChunk / 2; ++i) asm volatile("" : "+v"(a[i]));
    }
};
template <> struct Chunk<__half> {
    uint32_t p[kSeqChunk];            // address << 16 | weight
    __device__ __forceinline__ void set(int i, __half v, uint32_t addr) {
        p[i] = (addr << 16) | __half_as_ushort(v);
    }
    __device__ __forceinline__ float weight(int i) const {
        return __half2float(__ushort_as_half(uint16_t(p[i])));
    }
    __device__ __forceinline__ uint32_t addr(int i) const { return p[i] >> 16; }
    __device__ __forceinline__ void opaque() {
#pragma unroll
        for (int i = 0; i < kSeqChunk; ++i) asm volatile("" : "+v"(p[i]));
    }
};

template <int CPG> struct alignas(CPG * 4) HVec { float e[CPG]; };

// Place of a lane among the 16 lanes that a 16-byte LDS read serves together: lanes 0-3,
// 12-15, 20-23 and 24-27 of each half wave are one such set, the others another.
__device__ __forceinline__ int lds_place(int lane) {
    // of the eight quads of lanes in a half wave: 0 3 5 6 are one set, 1 2 4 7 the other
    // so each set has one quad of every pair (0 1) (2 3) (4 5) (6 7): its place in the set
    return ((lane >> 3) & 3) * 4 + (lane & 3);
}

// Weights k0 .. k0 + 15 of a row (first slot r0, nblk weights, block size 2^lb).  Their
// columns are random, so lanes that gather together would meet in the 64 LDS banks, 16
// columns of four floats wide.  The order inside a chunk is free: slot i takes, where
// there is one, a weight whose column is (i + the lane's place) mod 16, and the others
// fill the rest, so that most of the lanes served together read different banks.  The
// place is that of the chunk's number among its member's, whoever does the sum.
template <typename Tw, int CPG>
__device__ __forceinline__ void load_chunk(Chunk<Tw> &c, const Tw *__restrict__ values,
                                           const uint8_t *__restrict__ offsets, int64_t r0,
                                           int nblk, int lb, int k0, int H, int place) {
    static_assert(kSeqChunk == 16, "a slot per column class");
    Tw w[kSeqChunk];
    int col[kSeqChunk];
#pragma unroll
    for (int i = 0; i < kSeqChunk; ++i) {
        const int k = k0 + i;
        const bool ok = k < nblk;
        const int kc = ok ? k : nblk - 1;
        const Tw wi = values[r0 + kc];
        w[i] = ok ? wi : Tw(0.0f);
        const int cc = (kc << lb) + int(offsets[r0 + kc]);
        col[i] = ok ? (cc < H ? cc : H - 1) : H;        // the encode gives cc < H
    }
    // bits 4i .. 4i + 3 of `slot`: the weight that slot i takes; `taken`, `filled`: masks
    uint64_t slot = 0;
    uint32_t taken = 0, filled = 0;
#pragma unroll
    for (int i = 0; i < kSeqChunk; ++i) {
        const int s = (col[i] - place) & 15;
        if (!((filled >> s) & 1u)) {
            filled |= 1u << s;
            taken |= 1u << i;
            slot |= uint64_t(i) << (4 * s);
        }
    }
#pragma unroll
    for (int i = 0; i < kSeqChunk; ++i) {
        if (!((taken >> i) & 1u)) {
            const int s = __ffs(int(~filled)) - 1;
            filled |= 1u << s;
            slot |= uint64_t(i) << (4 * s);
        }
    }
#pragma unroll
    for (int s = 0; s < kSeqChunk; ++s) {
        const uint32_t from = uint32_t(slot >> (4 * s)) & 15u;
        Tw ws = w[0];
        int cs = col[0];
#pragma unroll
        for (int i = 1; i < kSeqChunk; ++i) {
            ws = from == uint32_t(i) ? w[i] : ws;
            cs = from == uint32_t(i) ? col[i] : cs;
        }
        c.set(s, ws, uint32_t(cs) * uint32_t(CPG * 4));
    }
}

template <typename Tw, int CPG>
__device__ __forceinline__ HVec<CPG> chunk_sum(const Chunk<Tw> &c, const char *hs) {
    HVec<CPG> acc;
#pragma unroll
    for (int q = 0; q < CPG; ++q) acc.e[q] = 0.0f;
    constexpr int kBatch = 8;                               // LDS reads in flight
#pragma unroll
    for (int i0 = 0; i0 < kSeqChunk; i0 += kBatch) {
        HVec<CPG> hv[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            hv[i] = *reinterpret_cast<const HVec<CPG> *>(hs + c.addr(i0 + i));
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const float w = c.weight(i0 + i);
#pragma unroll
            for (int q = 0; q < CPG; ++q) acc.e[q] = fmaf(w, hv[i].e[q], acc.e[q]);
        }
    }
    return acc;
}

// The cell of lstm_cell.h with its gates' activations apart, so that four lanes can take
// one each.
__device__ __forceinline__ float seq_activation(float z, bool candidate) {
    const float s = lstm_sigmoid(z), t = lstm_tanh(z);
    return candidate ? t : s;
}
__device__ __forceinline__ float seq_cell(float i, float f, float g, float o, float &c) {
    c = fmaf(f, c, i * g);
    return o * lstm_tanh(c);
}

// value of lane SRC (0..3) of the caller's aligned four lanes
template <int SRC> __device__ __forceinline__ float quad_lane(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
               0, __builtin_bit_cast(int, v), SRC * 0x55, 0xF, 0xF, false));
}

template <typename Tw, int CPG, int kItems>
__global__ __launch_bounds__(kSeqThreads) void lstm_seq_kernel(SeqArgs A) {
    constexpr int kRes = seq_resident(CPG);
    const int group = int(blockIdx.x) % kSeqXcds;
    const int member = int(blockIdx.x) / kSeqXcds;
    if (group >= A.groups) return;
    const int H = A.H;
    const int u0 = member * A.units;
    const int nu = H - u0 < A.units ? H - u0 : A.units;      // >= 1 by the launch
    const int rows = 4 * nu;                                 // row = 4 * unit + gate
    const int n0 = group * CPG;
    const int tid = int(threadIdx.x);
    const int lane = tid & (kWave - 1);
    const int wave = wave_uniform_i(tid / kWave);

    extern __shared__ __align__(16) char lds[];
    char *hs = lds;                                          // [H + 1][CPG], the last zero
    float *part = reinterpret_cast<float *>(lds + ((size_t(H + 1) * CPG * 4 + 15) & ~size_t(15)));
    int64_t *row_at = reinterpret_cast<int64_t *>(part + kSeqThreads * kRes * CPG);
    int *cbeg = reinterpret_cast<int *>(row_at + kSeqMaxRows);   // [kSeqMaxRows + 1]
    int *wtot = cbeg + kSeqMaxRows + 1;                      // [waves]
    int *bad = wtot + kSeqThreads / kWave;
    int *far = bad + 1;
    float *cst = reinterpret_cast<float *>(far + 1);         // [nu * CPG] cell state

    const Tw *values = static_cast<const Tw *>(A.values);
    // the member's rows: first slot and block size, and the first chunk of each
    int64_t info = 0;
    int nc = 0;
    if (tid < rows) {
        info = A.rowinfo[int64_t(tid & 3) * H + u0 + (tid >> 2)];
        const int lb = int(info & 0xFF);
        const int nblk = (H + (1 << lb) - 1) >> lb;
        nc = (nblk + kSeqChunk - 1) / kSeqChunk;
        row_at[tid] = info;
    }
    int incl = nc;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += o;
    }
    if (lane == kWave - 1) wtot[wave] = incl;
    if (tid == 0) *bad = 0;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wtot[w];
    cbeg[tid + 1] = before + incl;
    if (tid == 0) cbeg[0] = 0;
    for (int i = tid; i < nu * CPG; i += kSeqThreads) {
        const int n = n0 + i % CPG;
        cst[i] = n < A.batch ? A.c0[int64_t(u0 + i / CPG) * A.batch + n] : 0.0f;
    }
    if (tid < CPG) reinterpret_cast<float *>(hs)[H * CPG + tid] = 0.0f;
    __syncthreads();
    const int chunks = cbeg[rows];

    // chunk -> (first slot, weights, log2 b, first weight): the row whose chunks hold it
    auto fetch = [&](Chunk<Tw> &c, int id) {
        int lo = 0, hi = rows;                               // cbeg[lo] <= id < cbeg[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (cbeg[mid] <= id) lo = mid;
            else hi = mid;
        }
        const int64_t at = row_at[lo];
        const int lb = int(at & 0xFF);
        load_chunk<Tw, CPG>(c, values, A.offsets, at >> 8, (H + (1 << lb) - 1) >> lb, lb,
                            (id - cbeg[lo]) * kSeqChunk, H, lds_place(id & (kWave - 1)));
    };
    const int64_t slot_words = int64_t(A.groups) * H * CPG;
    uint32_t *ring = A.ring + int64_t(group) * H * CPG;
    const int words = H * CPG;
    const int items = rows * CPG;                            // (unit, column, gate)

    // the input products of step t, (unit, column, gate) by thread
    float ug[kItems] = {}, ug_next[kItems] = {};
    const uint32_t ldu = uint32_t(A.ldu);                    // all offsets fit 32 bits
    auto load_u = [&](int t, float (&u)[kItems]) {
        const float *at = A.U + int64_t(t) * A.batch;        // uniform
#pragma unroll
        for (int s = 0; s < kItems; ++s) {
            const int it = tid + s * kSeqThreads;
            const int n = n0 + (it >> 2) % CPG;
            const bool in = it < items && n < A.batch;       // others read a valid element
            u[s] = at[in ? uint32_t((it & 3) * H + u0 + (it >> 2) / CPG) * ldu + uint32_t(n) : 0u];
        }
    };
    load_u(0, ug_next);

    // Whether the whole group runs on one XCD: each member publishes its XCD's number and
    // reads the others' (in the slot of h_2, which its owners reset before any h_2).
    {
        uint32_t *at = ring + 2 * slot_words;
        const uint32_t mine = __builtin_amdgcn_s_getreg(kXccId);
        if (tid == 0)
            __hip_atomic_store(at + member, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool other = false;
        if (tid < A.members) {
            uint32_t v = kSentinel;
            for (uint32_t polls = 0; v == kSentinel && polls < A.max_polls; ++polls)
                v = __hip_atomic_load(at + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            other = v != mine;                               // so is one that never came
        }
        if (tid == 0) *far = 0;
        __syncthreads();
        if (other) *far = 1;
        __syncthreads();
    }
    const bool near = *far == 0 && A.far == 0u;              // uniform
    // A word of the ring.  On one XCD a plain store puts it where the readers look, the
    // L2 that they share (the vector caches write through); a device-scope store writes
    // it to memory and costs the readers a round trip to there (measured: 1.0 instead of
    // 1.8 us from the store to the last member's read).
    auto publish = [&](uint32_t *base, uint32_t i, uint32_t v) {
        if (near)
            __hip_atomic_store(base + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_store(base + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // the member's chunks, in registers for the whole sequence (the launch's rule: they fit)
    Chunk<Tw> res[kRes];
#pragma unroll
    for (int j = 0; j < kRes; ++j) {
        const int id = tid + j * kSeqThreads;
        fetch(res[j], id < chunks ? id : chunks - 1);
    }
    for (int t = 0; t < A.T; ++t) {
#pragma unroll
        for (int s = 0; s < kItems; ++s) ug[s] = ug_next[s];
        // h_{t-1} into LDS
        if (t == 0) {
            for (int i = tid; i < words; i += kSeqThreads) {
                const int n = n0 + i % CPG;
                reinterpret_cast<float *>(hs)[i] =
                    n < A.batch ? A.h0[int64_t(i / CPG) * A.batch + n] : 0.0f;
            }
        } else {
            // 8 bytes at a time (words is even: H or CPG is)
            const uint64_t *src = reinterpret_cast<const uint64_t *>(
                ring + int64_t((t - 1) % 3) * slot_words);
            uint64_t *dst = reinterpret_cast<uint64_t *>(hs);
            constexpr int kBatch = 4;
            uint32_t polls = 0;
            for (int i0 = tid; i0 < words / 2; i0 += kBatch * kSeqThreads) {
                uint64_t v[kBatch];
                for (;;) {
                    bool wait = false;
#pragma unroll
                    for (int b = 0; b < kBatch; ++b) {
                        const int i = i0 + b * kSeqThreads;
                        v[b] = __hip_atomic_load(src + uint32_t(i < words / 2 ? i : i0),
                                                 __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int b = 0; b < kBatch; ++b)
                        wait = wait || uint32_t(v[b]) == kSentinel ||
                               uint32_t(v[b] >> 32) == kSentinel;
                    if (!wait) break;
                    // over the limit for this step, or another member is
                    ++polls;
                    if (polls >= A.max_polls ||
                        ((polls & 63u) == 0 && __hip_atomic_load(A.failed, __ATOMIC_RELAXED,
                                                                 __HIP_MEMORY_SCOPE_AGENT))) {
                        *bad = 1;
                        break;
                    }
                }
#pragma unroll
                for (int b = 0; b < kBatch; ++b) {
                    const int i = i0 + b * kSeqThreads;
                    if (i < words / 2) dst[i] = v[b];
                }
            }
        }
        __syncthreads();
        if (*bad) {                                          // uniform: same value for all
            if (tid == 0)
                __hip_atomic_store(A.failed, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        // every member has finished with h_{t-2} (at step 1: with the XCD numbers): its
        // slot takes h_{t+1} next
        if (t >= 1) {
            uint32_t *old = ring + int64_t((t + 1) % 3) * slot_words;
            for (int it = tid; it < items; it += kSeqThreads)
                if ((it & 3) == 0)
                    publish(old, uint32_t(u0 * CPG + (it >> 2)), kSentinel);
        }
#pragma unroll
        for (int j = 0; j < kRes; ++j) {
            const int id = j * kSeqThreads + tid;
            if (j * kSeqThreads + wave * kWave < chunks) {   // wave-uniform
                res[j].opaque();
                const HVec<CPG> acc = chunk_sum<Tw, CPG>(res[j], hs);
                if (id < chunks) *reinterpret_cast<HVec<CPG> *>(part + id * CPG) = acc;
            }
        }
        // the sentinel's stores are acknowledged (long ago) before h_t goes out, and the
        // next step's input products set out: they are back before the next poll, which
        // would wait for them (loads return in order)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        load_u(t + 1 < A.T ? t + 1 : t, ug_next);
        __syncthreads();
        // a row's chunks in ascending order, four lanes (one per gate) to a unit
        float sum[kItems];
#pragma unroll
        for (int s = 0; s < kItems; ++s) {
            sum[s] = 0.0f;
            const int it = tid + s * kSeqThreads;
            if (it < items) {
                const int cell = it >> 2;
                const int r = (cell / CPG) * 4 + (it & 3);
                const int b = cbeg[r], e = cbeg[r + 1];
                const float *p = part + (cell % CPG);
                for (int k = b; k < e; k += 8) {             // 8 loads in flight
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = p[(k + i < e ? k + i : e - 1) * CPG];
#pragma unroll
                    for (int i = 0; i < 8; ++i) sum[s] += k + i < e ? v[i] : 0.0f;
                }
            }
        }
#pragma unroll
        for (int s = 0; s < kItems; ++s) {
            const int it = tid + s * kSeqThreads;
            if (it - lane < items) {                         // wave-uniform: DPP below
                const float z = sum[s] + ug[s];
                const int cell = it >> 2;
                // each lane its own gate's activation, then all four the unit's cell
                const float act = seq_activation(z, (it & 3) == 2);
                float c = cst[cell < nu * CPG ? cell : 0];
                const float h = seq_cell(quad_lane<0>(act), quad_lane<1>(act),
                                         quad_lane<2>(act), quad_lane<3>(act), c);
                if (it < items && (it & 3) == 0) {
                    cst[cell] = c;
                    uint32_t bits = __builtin_bit_cast(uint32_t, h);
                    if (bits == kSentinel) bits = 0x7FC00000u;     // any NaN will do
                    publish(ring + int64_t(t % 3) * slot_words, uint32_t(u0 * CPG + cell), bits);
                    const int n = n0 + cell % CPG;
                    if (n < A.batch)
                        (A.h_seq + int64_t(t) * A.batch)[uint32_t(u0 + cell / CPG) * ldu +
                                                         uint32_t(n)] =
                            __builtin_bit_cast(float, bits);
                }
            }
        }
    }
    // the final cell state waits in the one slot that nobody reads any more (h_{T-2} is in
    // slot (T-2) % 3 and h_{T-1} in (T-1) % 3); the initial state stays as it was
    __syncthreads();
    uint32_t *out = ring + int64_t(A.T % 3) * slot_words + u0 * CPG;
    for (int i = tid; i < nu * CPG; i += kSeqThreads)
        out[i] = __builtin_bit_cast(uint32_t, cst[i]);
}

// 1 while a sequence of this process has its turn on the device.
__device__ uint32_t seq_turn;

// The sentinel into every slot, no failure, and the turn: one lane waits for it while the
// holder runs to its end.  The wait is bounded too; without the turn the sequence is still
// right, since its members' waits are bounded, only slower if another has the CUs.
__global__ __launch_bounds__(256) void lstm_seq_init_kernel(uint32_t *ring, int64_t words,
                                                            uint32_t *failed) {
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < words;
         i += int64_t(gridDim.x) * 256)
        ring[i] = kSentinel;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        failed[0] = 0u;
        uint32_t mine = 0u;
        for (uint32_t polls = 0; polls < kTurnPolls; ++polls) {
            if (atomicCAS(&seq_turn, 0u, 1u) == 0u) {
                mine = 1u;
                break;
            }
            __builtin_amdgcn_s_sleep(32);
        }
        failed[1] = mine;
    }
}

// The turn goes back (by the holder alone).
__device__ __forceinline__ void seq_turn_over(const SeqArgs &A) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && A.failed[1] != 0u)
        __hip_atomic_store(&seq_turn, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The final state into the caller's buffers.  After a failure: the whole sequence of batch
// column blockIdx.x by this workgroup alone, with the sums in lstm_seq_kernel's order: a
// lane per chunk, the chunks' sums added in ascending order.  The rows of a block-size
// group are equally long and follow each other in storage order, so a wave takes as many of
// them as it has lanes for their chunks.  Bound: the instructions that order a chunk.
// H = 1024, T = 200, batch 32, fp16, 5 %: 40 ms, and 504 with a wave per row; the
// sequence that did not fail takes 0.6.
template <typename Tw>
__global__ __launch_bounds__(kFinishThreads) void lstm_finish_kernel(
    SeqArgs A, int cpg, const int32_t *__restrict__ perm, BinTable bins) {
    extern __shared__ __align__(16) char lds[];
    const int n = int(blockIdx.x);
    const int tid = int(threadIdx.x);
    const int H = A.H;
    if (A.failed[0] == 0u) {                                 // uniform
        seq_turn_over(A);                                    // every member has left
        const uint32_t *c = A.ring + int64_t(A.T % 3) * A.groups * H * cpg +
                            int64_t(n / cpg) * H * cpg + n % cpg;
        for (int u = tid; u < H; u += kFinishThreads) {
            A.c_out[int64_t(u) * A.batch + n] = __builtin_bit_cast(float, c[u * cpg]);
            A.h_out[int64_t(u) * A.batch + n] =
                A.h_seq[int64_t(u) * A.ldu + int64_t(A.T - 1) * A.batch + n];
        }
        return;
    }
    const Tw *values = static_cast<const Tw *>(A.values);
    float *h = reinterpret_cast<float *>(lds);               // [H + 1], the last zero
    float *c = h + H + 1;                                    // [H]
    float *z = c + H;                                        // [4H]
    uint16_t *fc = reinterpret_cast<uint16_t *>(z + 4 * H);  // [4H]
    for (int u = tid; u < H; u += kFinishThreads) {
        h[u] = A.h0[int64_t(u) * A.batch + n];
        c[u] = A.c0[int64_t(u) * A.batch + n];
    }
    if (tid == 0) h[H] = 0.0f;
    const int lane = tid & (kWave - 1);
    const int wave = wave_uniform_i(tid / kWave);
    // the number of each row's first chunk among its member's
    if (tid < A.members) {
        int first = 0;
        for (int u = tid * A.units; u < H && u < (tid + 1) * A.units; ++u)
            for (int g = 0; g < 4; ++g) {
                fc[4 * u + g] = uint16_t(first);
                const int lb = int(A.rowinfo[int64_t(g) * H + u] & 0xFF);
                first += (((H + (1 << lb) - 1) >> lb) + kSeqChunk - 1) / kSeqChunk;
            }
    }
    for (int t = 0; t < A.T; ++t) {
        __syncthreads();
        for (int g = 0; g < bins.nbins; ++g) {               // uniform
            const int lb = bins.log2b[g];
            const int nblk = int(bins.nblk[g]);
            const int nc = (nblk + kSeqChunk - 1) / kSeqChunk;     // <= 64
            const int lgL = nc <= 1 ? 0 : 32 - __builtin_clz(nc - 1);
            const int rows = int(bins.rows[g]);
            const int per_wave = kWave >> lgL;
            const int in_row = lane & ((1 << lgL) - 1);
            const int id = in_row < nc ? in_row : nc - 1;
            for (int i0 = wave * per_wave; i0 < rows; i0 += kFinishThreads / kWave * per_wave) {
                const int i = i0 + (lane >> lgL);            // uniform bounds: shuffles below
                const int ic = i < rows ? i : rows - 1;
                const int r = perm[bins.first_row[g] + ic];
                const int64_t first = bins.first_elem[g] + int64_t(ic) * nblk;
                Chunk<Tw> ch;
                load_chunk<Tw, 1>(ch, values, A.offsets, first, nblk, lb, id * kSeqChunk, H,
                                  lds_place((fc[4 * (r % H) + r / H] + id) & (kWave - 1)));
                const HVec<1> acc = chunk_sum<Tw, 1>(ch, lds);
                float sum = 0.0f;
                for (int k = 0; k < nc; ++k)
                    sum += __shfl(acc.e[0], (lane - in_row) + k, kWave);
                if (i < rows && in_row == 0)
                    z[r] = sum + A.U[int64_t(r) * A.ldu + int64_t(t) * A.batch + n];
            }
        }
        __syncthreads();
        for (int u = tid; u < H; u += kFinishThreads) {
            float cu = c[u];
            const float hn =
                seq_cell(seq_activation(z[u], false), seq_activation(z[H + u], false),
                         seq_activation(z[2 * H + u], true), seq_activation(z[3 * H + u], false), cu);
            c[u] = cu;
            h[u] = hn;
            A.h_seq[int64_t(u) * A.ldu + int64_t(t) * A.batch + n] = hn;
        }
    }
    for (int u = tid; u < H; u += kFinishThreads) {          // this thread's own units
        A.h_out[int64_t(u) * A.batch + n] = h[u];
        A.c_out[int64_t(u) * A.batch + n] = c[u];
    }
    seq_turn_over(A);        // only now: these workgroups held CUs that the next one needs
}

struct SeqPlan {
    int cpg, groups, members, units;
    size_t lds, finish_lds;
};

// Whether and how the sequence runs as one launch.  Columns per group: the fewest that
// leave at most 8 groups.
bool seq_plan(const darb_plan &whh, int64_t H, int64_t T, int64_t batch, SeqPlan &p) {
    // setting up (the tables, the registers, two more launches) costs about as much as 8
    // to 11 steps save.  A layer of 16 steps, us, this way and with a launch per step, batch
    // 1 / 8 / 16 / 64: H = 128 52 / 54 / 57 / 60 and 78 / 85 / 87 / 91, H = 1024 66 / 73 /
    // 80 / 136 and 92 / 109 / 116 / 203
    if (T < 16 || batch > 64 || H < 16 || T > 0x7FFFFFFF) return false;
    // one workgroup per CU, an XCD's 32 for each group
    if (whh.cus < kSeqXcds * kSeqMembers) return false;
    for (int g = 0; g < whh.bins.nbins; ++g)
        if (whh.bins.nblk[g] > kSeqMaxNblk) return false;
    p.cpg = batch <= 8 ? 1 : batch <= 16 ? 2 : batch <= 32 ? 4 : 8;
    if (p.cpg == 1 && H % 2 != 0) p.cpg = 2;              // h is read 8 bytes at a time
    p.groups = int((batch + p.cpg - 1) / p.cpg);
    // h's addresses in LDS are kept in 16 bits
    if ((H + 1) * p.cpg * 4 > 65536) return false;
    p.units = int(lstm_units(H));
    p.members = int((H + p.units - 1) / p.units);
    // a member's rows have a thread each, its (row, column) sums at most two per thread
    if (4 * p.units > kSeqMaxRows || 4 * p.units * p.cpg > 2 * kSeqThreads) return false;
    // every member's weights stay in its registers: a form that read those past them again
    // at each step took 33 us a step (H = 1500, batch 20, fp16, 6.5 % kept, 10 of 32 members
    // past the limit) and 50 us (H = 2048, batch 32, 5 %), a launch per step 11.6 and 14.4
    if (whh.lstm_chunks > seq_resident(p.cpg) * kSeqThreads) return false;
    // the kernels' 32-bit offsets into the input products
    if (4 * H * T * batch >= (int64_t(1) << 30)) return false;
    // the ring and the flags live in the workspace's last 4 * H * batch floats
    if (3 * H * p.groups * p.cpg + 16 > 4 * H * batch) return false;
    const size_t hs = (size_t(H + 1) * p.cpg * 4 + 15) & ~size_t(15);
    p.lds = hs + size_t(kSeqThreads) * seq_resident(p.cpg) * p.cpg * 4 + size_t(kSeqMaxRows) * 8 +
            (kSeqMaxRows + 1 + kSeqThreads / kWave + 2) * 4 + size_t(p.units) * p.cpg * 4;
    p.finish_lds = size_t(8 * H + 1) * 4;
    return int64_t(p.lds) <= kSeqMaxLds && int64_t(p.finish_lds) <= kSeqMaxLds;
}

// A call's three launches follow each other without another call's between them: on
// streams that share a hardware queue, a wait for the turn in between would hold up the
// launch that gives it back.
std::mutex launch_order;

template <typename Tw>
hipError_t launch_seq_t(const darb_plan &whh, const SeqPlan &p, const SeqArgs &a, hipStream_t s) {
    const int64_t words = int64_t(3) * p.groups * a.H * p.cpg;
    const int64_t init = (words + 255) / 256 < 256 ? (words + 255) / 256 : 256;
    std::lock_guard<std::mutex> lock(launch_order);
    hipLaunchKernelGGL(lstm_seq_init_kernel, dim3(unsigned(init)), dim3(256), 0, s, a.ring, words,
                       a.failed);
    const dim3 grid(unsigned(kSeqXcds * p.members));
    const bool one = 4 * p.units * p.cpg <= kSeqThreads;
#define DARB_SEQ(C)                                                                          \
    do {                                                                                     \
        if (one)                                                                             \
            hipLaunchKernelGGL((lstm_seq_kernel<Tw, C, 1>), grid, dim3(kSeqThreads), p.lds,   \
                               s, a);                                                         \
        else                                                                                  \
            hipLaunchKernelGGL((lstm_seq_kernel<Tw, C, 2>), grid, dim3(kSeqThreads), p.lds,   \
                               s, a);                                                         \
    } while (0)
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;                // nothing was launched
    switch (p.cpg) {
        case 1: DARB_SEQ(1); break;
        case 2: DARB_SEQ(2); break;
        case 4: DARB_SEQ(4); break;
        default: DARB_SEQ(8); break;
    }
#undef DARB_SEQ
    e = hipGetLastError();
    // also after an error: it gives the turn back
    hipLaunchKernelGGL((lstm_finish_kernel<Tw>), dim3(unsigned(a.batch)), dim3(kFinishThreads),
                       p.finish_lds, s, a, p.cpg, whh.d_perm, whh.bins);
    const hipError_t last = hipGetLastError();
    return e != hipSuccess ? e : last;
}

}  // namespace

bool lstm_seq_applies(const darb_plan &whh, int64_t H, int64_t T, int64_t batch, hipStream_t s) {
    SeqPlan p;
    if (!seq_plan(whh, H, T, batch, p)) return false;
    // not into a graph: branches that share a hardware queue may place a wait for the turn
    // before the launch that gives it back
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st == hipStreamCaptureStatusNone;
}

hipError_t launch_lstm_seq(const darb_plan &whh, int wdtype, const void *values,
                           const uint8_t *offsets, int64_t H, int64_t T, int64_t batch,
                           const float *U, float *scratch, float *h_seq, float *h, float *c,
                           uint32_t max_polls, bool far, hipStream_t s) {
    SeqPlan p;
    if (!seq_plan(whh, H, T, batch, p)) return hipErrorInvalidConfiguration;
    SeqArgs a{};
    a.values = values;
    a.offsets = offsets;
    a.rowinfo = whh.d_rowinfo;
    a.U = U;
    a.h0 = h;
    a.c0 = c;
    a.h_seq = h_seq;
    a.h_out = h;
    a.c_out = c;
    a.ring = reinterpret_cast<uint32_t *>(scratch);
    a.failed = a.ring + 3 * int64_t(p.groups) * H * p.cpg;
    a.ldu = T * batch;
    a.H = int32_t(H);
    a.T = int32_t(T);
    a.batch = int32_t(batch);
    a.groups = p.groups;
    a.members = p.members;
    a.units = p.units;
    a.max_polls = max_polls;
    a.far = far ? 1u : 0u;
    if (wdtype == DARB_F32) return launch_seq_t<float>(whh, p, a, s);
    return launch_seq_t<__half>(whh, p, a, s);
}

}  // namespace darb

int darb_test_lstm_seq(const darb_plan *whh, int wdtype, const void *values,
                       const uint8_t *offsets, int64_t H, int64_t T, int64_t batch,
                       const float *U, float *scratch, float *h_seq, float *h, float *c,
                       uint32_t max_polls, int far, void *stream) {
    return int(darb::launch_lstm_seq(*whh, wdtype, values, offsets, H, T, batch, U, scratch,
                                     h_seq, h, c, max_polls, far != 0,
                                     static_cast<hipStream_t>(stream)));
}

int64_t darb_test_lstm_chunks(const darb_plan *whh) { return whh->lstm_chunks; }

int darb_test_lstm_seq_applies(const darb_plan *whh, int64_t H, int64_t T, int64_t batch,
                               void *stream) {
    return darb::lstm_seq_applies(*whh, H, T, batch, static_cast<hipStream_t>(stream)) ? 1 : 0;
}
