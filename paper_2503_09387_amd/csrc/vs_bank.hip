// Memory bank of the semantic carriers (VideoScan Section 3.3, memory mechanism): at most M
// carriers are kept; when one arrives at a full bank, embeddings of adjacent carriers are
// compared and the older carrier of the most similar pair is dropped.  Reading of the passage:
// the sequence bank[0..M-1], incoming has M adjacent pairs (i, i+1); victim = the i with the
// largest cosine, of equal ones the smallest i (policy 1: the i whose cosine with the incoming
// carrier is largest).  A vector of norm 0 has cosine 0 with everything.
//
// Two steps on the device, no host round trip in between:
//   1. bank_cosine_kernel: one workgroup per pair, fp64 sums in a fixed order (the products of
//      bf16 or fp32 values are exact in fp64, so the cosines agree with a plain fp64 evaluation
//      to ~1e-13 and the victim is the same unless two cosines are that close);
//   2. bank_shift_kernel: every workgroup finds the victim from the M cosines (or reads the
//      index an earlier call left in device memory), then a table of per-carrier rows (the
//      embeddings, or one layer's K or V rows) drops that row, closes the gap and takes the
//      new row last.  A workgroup owns a 128-byte wide column block of one table: it loads up to
//      256 rows into registers, waits for all its wavefronts to have theirs, and stores them one
//      row up, so the move is in place and takes one round trip per 256 rows.  (The rate of a
//      compute unit bounds it: 1 KB wide blocks left 7 workgroups for the embeddings and 56 for the
//      rows of 28 layers, 9.3 us per launch on average at M = 128; these take 4.3 us.)
#include "vs_internal.h"

namespace vs {
namespace {

constexpr int kShiftThreads = 256;
constexpr int kShiftLanes = 8;                             // 16-byte pieces of a row side by side: a column block of 128 bytes
constexpr int kShiftRows = kShiftThreads / kShiftLanes;    // rows per step
constexpr int kShiftSteps = 8;                             // rows per thread and pass: 256 rows per pass
constexpr int kShiftPass = kShiftRows * kShiftSteps;

__device__ __forceinline__ double block_sum(double x, double* lds) {  // fixed order, every thread gets the sum
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) lds[w] = x;
    __syncthreads();
    return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// Bound by the trips to memory: both rows are requested at once, 16 bytes per thread, and pass through
// LDS, from where thread t takes the elements t, t + 256, .. in order (7.0 -> 4.3 us at 128 x 3584).  A short row is
// read in that order right away (a push at 128 rows, this way and through LDS: 256 wide 6.4 and 6.8 us, 512 6.6 and 6.8, 1024 6.75
// and 6.73).
constexpr int kShortRow = 512;
template <typename T>
__global__ __launch_bounds__(256) void bank_cosine_kernel(const T* __restrict__ e, const T* __restrict__ e_new,
                                                          int M, int d, int policy, double* __restrict__ cosines) {
    constexpr int kVec = 16 / sizeof(T), kSeg = 512 * kVec;  // elements of a row in LDS at a time: 8 KB
    __shared__ __attribute__((aligned(16))) T rows[2][kSeg];
    __shared__ double lds[4];
    const int i = blockIdx.x;
    const T* a = e + (int64_t)i * d;
    const T* b = (policy == 1 || i + 1 == M) ? e_new : e + (int64_t)(i + 1) * d;
    double ab = 0.0, aa = 0.0, bb = 0.0;
    if (d <= kShortRow) {
        for (int j = threadIdx.x; j < d; j += 256) {
            const double x = (double)to_f32(a[j]), y = (double)to_f32(b[j]);
            ab += x * y;
            aa += x * x;
            bb += y * y;
        }
    } else for (int j0 = 0; j0 < d; j0 += kSeg) {
        const int n = min(kSeg, d - j0), n16 = n / kVec;  // (rows are whole multiples of 16 bytes)
        raw16 va[2], vb[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = min((int)threadIdx.x + 256 * u, n16 - 1);
            va[u] = reinterpret_cast<const raw16*>(a + j0)[c];
            vb[u] = reinterpret_cast<const raw16*>(b + j0)[c];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            keep_here(va[u]);
            keep_here(vb[u]);
        }
        if (j0) __syncthreads();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = threadIdx.x + 256 * u;
            if (c < n16) {
                reinterpret_cast<raw16*>(rows[0])[c] = va[u];
                reinterpret_cast<raw16*>(rows[1])[c] = vb[u];
            }
        }
        __syncthreads();
#pragma unroll 4
        for (int j = threadIdx.x; j < n; j += 256) {
            const double x = (double)to_f32(rows[0][j]), y = (double)to_f32(rows[1][j]);
            ab += x * y;
            aa += x * x;
            bb += y * y;
        }
    }
    ab = block_sum(ab, lds);
    aa = block_sum(aa, lds);
    bb = block_sum(bb, lds);
    if (threadIdx.x == 0) cosines[i] = (aa > 0.0 && bb > 0.0) ? ab / (sqrt(aa) * sqrt(bb)) : 0.0;
}

struct ShiftTables {
    char* base[kBankMaxTables];           // table t: rows of row_bytes bytes
    const char* new_row[kBankMaxTables];  // the row that becomes the last one
};

struct ShiftParams {
    ShiftTables t;
    int64_t row_bytes;
    int first;              // rows in front of the carriers
    int M;                  // carriers of a full bank
    int append_at;          // >= 0: room left, the new row goes to first + append_at; -1: drop the victim
    const double* cosines;  // [M], or null: the victim's index is read from victim_io
    int* victim_io;         // device int (may be null when cosines are given)
};

__global__ __launch_bounds__(kShiftThreads) void bank_shift_kernel(ShiftParams p) {
    __shared__ int s_victim;
    __shared__ double s_cos[kShiftThreads / 64];
    __shared__ int s_idx[kShiftThreads / 64];
    const int tid = threadIdx.x;
    const int64_t col = (int64_t)blockIdx.x * (16 * kShiftLanes) + (tid % kShiftLanes) * 16;  // this thread's 16 bytes of a row
    const int lr = tid / kShiftLanes;
    char* const base = p.t.base[blockIdx.y] + (int64_t)p.first * p.row_bytes;
    const char* const new_row = p.t.new_row[blockIdx.y];
    const bool in_row = col < p.row_bytes;
    if (p.append_at >= 0) {
        if (lr == 0 && in_row)
            *reinterpret_cast<uint4*>(base + (int64_t)p.append_at * p.row_bytes + col) =
                *reinterpret_cast<const uint4*>(new_row + col);
        if (p.victim_io && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *p.victim_io = -1;
        return;
    }
    int victim;
    if (p.cosines) {
        // largest cosine, of equal ones the smallest index: thread t looks at cosines t, t + 256, ..,
        // the candidates of a wavefront meet by lane exchanges, those of the wavefronts in LDS
        double best_cos = 0.0;
        int best = 0x7fffffff;  // (none yet)
        for (int i = tid; i < p.M; i += kShiftThreads) {
            const double c = p.cosines[i];
            if (best == 0x7fffffff || c > best_cos) {
                best = i;
                best_cos = c;
            }
        }
        auto better = [](double c_b, int i_b, double c_a, int i_a) {  // does candidate b beat candidate a?
            return i_b != 0x7fffffff && (i_a == 0x7fffffff || c_b > c_a || (c_b == c_a && i_b < i_a));
        };
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const double c_o = __shfl_xor(best_cos, off);
            const int i_o = __shfl_xor(best, off);
            if (better(c_o, i_o, best_cos, best)) {
                best_cos = c_o;
                best = i_o;
            }
        }
        if ((tid & 63) == 0) {
            s_cos[tid >> 6] = best_cos;
            s_idx[tid >> 6] = best;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w2 = 1; w2 < kShiftThreads / 64; ++w2)
                if (better(s_cos[w2], s_idx[w2], best_cos, best)) {
                    best_cos = s_cos[w2];
                    best = s_idx[w2];
                }
            s_victim = best;
        }
        __syncthreads();
        victim = s_victim;
        if (p.victim_io && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *p.victim_io = victim;
    } else {
        victim = *p.victim_io;
    }
    victim = min(max(victim, 0), p.M - 1);  // (an index from device memory is not trusted to be in range)
    // rows victim+1 .. M-1 move to victim .. M-2, kShiftPass rows per pass: all loads of a pass, a
    // barrier, all its stores (a later pass reads only rows that no earlier pass has written).  (Requesting the rows
    // before the victim is known saves no time, because the launch is as long as its longest workgroup either way, and
    // reads the rows in front of the victim for nothing: 28 layers of 128 rows of 1 KB, victim first / last, 4.1 / 2.4
    // us and 4.1 / 3.1 so, rows of 8 KB 20.1 / 3.6 and 19.8 / 11.5.)
    for (int r0 = victim; r0 + 1 < p.M; r0 += kShiftPass) {
        raw16 v[kShiftSteps];
#pragma unroll
        for (int u = 0; u < kShiftSteps; ++u) {  // destination rows (past the end: the last row, not stored)
            if (r0 + kShiftRows * u + 1 >= p.M) break;
            const int r = min(r0 + kShiftRows * u + lr + 1, p.M - 1);
            v[u] = *reinterpret_cast<const raw16*>(base + (int64_t)r * p.row_bytes + min(col, p.row_bytes - 16));
        }
#pragma unroll
        for (int u = 0; u < kShiftSteps; ++u) keep_here(v[u]);  // (this wavefront's rows are in registers)
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kShiftSteps; ++u) {
            const int r = r0 + kShiftRows * u + lr;
            if (r + 1 < p.M && in_row)
                *reinterpret_cast<raw16*>(base + (int64_t)r * p.row_bytes + col) = v[u];
        }
        __syncthreads();
    }
    if (lr == 0 && in_row)
        *reinterpret_cast<uint4*>(base + (int64_t)(p.M - 1) * p.row_bytes + col) = *reinterpret_cast<const uint4*>(new_row + col);
}

}  // namespace

hipError_t launch_bank_cosines(const void* e, const void* e_new, int32_t M, int32_t d, int32_t dtype,
                               int32_t policy, double* cosines, hipStream_t st) {
    if (dtype == VS_F32)
        bank_cosine_kernel<float><<<M, 256, 0, st>>>((const float*)e, (const float*)e_new, M, d, policy, cosines);
    else
        bank_cosine_kernel<__bf16><<<M, 256, 0, st>>>((const __bf16*)e, (const __bf16*)e_new, M, d, policy, cosines);
    return hipGetLastError();
}

hipError_t launch_bank_shift(int32_t n_tables, void* const* bases, const void* const* new_rows, int64_t row_bytes,
                             int32_t first, int32_t M, int32_t append_at, const double* cosines, int32_t* victim_io,
                             hipStream_t st) {
    for (int32_t t0 = 0; t0 < n_tables; t0 += kBankMaxTables) {
        const int32_t n = n_tables - t0 < kBankMaxTables ? n_tables - t0 : kBankMaxTables;
        ShiftParams p;
        for (int32_t t = 0; t < n; ++t) {
            p.t.base[t] = (char*)bases[t0 + t];
            p.t.new_row[t] = (const char*)new_rows[t0 + t];
        }
        p.row_bytes = row_bytes;
        p.first = first;
        p.M = M;
        p.append_at = append_at;
        p.cosines = cosines;
        p.victim_io = victim_io;
        bank_shift_kernel<<<dim3((unsigned)((row_bytes + 16 * kShiftLanes - 1) / (16 * kShiftLanes)), (unsigned)n), kShiftThreads, 0, st>>>(p);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace vs
