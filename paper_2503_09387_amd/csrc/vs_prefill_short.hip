// Frame prefill attention for bf16 storage on gfx950 over a SHORT key sequence (VideoScan Section 3.3,
// prefilling phase; Eq. 1 of Section 3.1): the start of a video, short questions.
//
// With few keys the general kernel (vs_prefill_mfma.hip) is all fixed cost: 128 query rows per workgroup
// leave too few workgroups, so the keys are split over several of them, whose partial results
// then meet through memory.  Here a workgroup owns 32 packed query rows (row = token * G + head, as there) of
// one KV head and ALL their keys, so nothing leaves it but the output:
//   * its four wavefronts share the keys: wavefront w takes the blocks of 32 keys w, w + 4, ..; each has
//     LDS buffers of its own (two stages of a K and a V block) and works without a barrier;
//   * K and V blocks and the query rows go from global memory straight into LDS, whole 256-byte rows
//     per 16 lanes, the 16-byte pieces of a row permuted by the row number so that the row-wise K and Q
//     reads and the transposing V reads are free of bank conflicts; the next block is under way
//     while one is worked on;
//   * S^T = K Q^T and O^T += V^T P^T with v_mfma_f32_32x32x16_bf16: a lane owns one query row's
//     column, the probabilities already are the B operand of the second product;
//   * the softmax reference is refreshed only when a score exceeds it by more than 2^8; row sums are
//     taken over the rounded probabilities;
//   * the four wavefronts' results (fp32) meet in LDS, each closing 32 of the 128 output dims.
// Every workgroup of a KV head reads all of the head's K and V through its compute unit, at ~60 KB/us (what a
// compute unit has under way, 32 KB, divided by the trip to L2): that is what bounds it and ends its range.
// The register budget is that of two wavefronts per SIMD, although one runs: with 512 registers the compiler keeps the sums
// in accumulation registers and copies all 64 out and back in every block (170 tokens over 430 rows 10.4 -> 9.4 us a
// launch, over 16 rows 6.6 -> 6.1).
#include "vs_internal.h"
#include "vs_prefill_map.h"

namespace vs {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int D = 128, kRowBytes = D * 2;
constexpr int kBlockBytes = 32 * kRowBytes;      // 32 keys (or query rows): 8 KB
constexpr int kStageBytes = 2 * kBlockBytes;     // K block, then V block
constexpr int kWaveLds = 2 * kStageBytes;        // two stages
constexpr int kWaves = 4, kThreads = 64 * kWaves;
constexpr int kLds = kWaves * kWaveLds + kBlockBytes + kWaves * 32 * 8;  // + query rows, + (reference, sum) per wavefront and row
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLazyMax = 8.0f;

struct ShortParams {
    const char* kc;
    const char* vc;
    const char* q;
    const char* kf;
    const char* vf;
    __bf16* out;
    char* k_append_dst;  // rows append_first .. T-1 of the run are copied here (null: none)
    char* v_append_dst;
    int append_first;
    int L, T, G, Hq, Hkv, M;
    int n_row_groups, units_per_xcd;
    float scale_log2e;
    QuickDiv by_G, by_row_groups;
};

__device__ __forceinline__ bf16x4 lds_read_tr(const char* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(p));
}

// 16 bytes per lane from global memory straight into LDS, lane i's at dst + 16 i (assembly: for the
// builtin form the compiler waits for all such loads before any LDS read); from a lane's own address,
// or eight in a row, 1 KB apart in LDS, from offsets of its own to an address that is the wavefront's (M0 is stepped
// between them: a wavefront alone on its SIMD takes 5 cycles for every instruction)
__device__ __forceinline__ void load_lds16x8(const char* base, const unsigned (&off)[8], unsigned dst) {
    asm volatile("s_mov_b32 m0, %[d]\n\ts_nop 4\n\t"
                 "global_load_lds_dwordx4 %[o0], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o1], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o2], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o3], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o4], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o5], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o6], %[b]\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
                 "global_load_lds_dwordx4 %[o7], %[b]"
                 :
                 : [d] "s"(dst), [b] "s"(base), [o0] "v"(off[0]), [o1] "v"(off[1]), [o2] "v"(off[2]), [o3] "v"(off[3]),
                   [o4] "v"(off[4]), [o5] "v"(off[5]), [o6] "v"(off[6]), [o7] "v"(off[7])
                 : "memory", "scc");
}
__device__ __forceinline__ void load_lds16(const char* src, unsigned dst) {
    asm volatile("s_mov_b32 m0, %[d]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[s], off" : : [d] "s"(dst), [s] "v"(src) : "memory");
}
#define VS_WAIT_LOADS(n) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(n) : "memory")

__global__ __launch_bounds__(kThreads, 2) void prefill_short_kernel(ShortParams p) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    // unit = (KV head, row group); ids of one residue modulo 8 (one XCD) take consecutive units, so that a
    // head's K and V are read into few L2s
    const int slot = (int)(blockIdx.x >> 3), unit = (int)(blockIdx.x & 7) * p.units_per_xcd + slot;
    if (unit >= p.n_row_groups * p.Hkv) return;  // spare ids (slot < units_per_xcd by the grid)
    const int g = __builtin_amdgcn_readfirstlane(div_by(unit, p.by_row_groups));
    const int row0 = (unit - g * p.n_row_groups) * 32;
    const int L = p.L, T = p.T, M = p.M, G = p.G;
    const int kv_row = p.Hkv * kRowBytes;
    // (all fetched at once; opaque, or the compiler turns a choice between two of them into a choice of
    // where in the argument block to load from)
    const char *kc = p.kc, *vc = p.vc, *kf = p.kf, *vf = p.vf, *qp = p.q;
    asm volatile("" : "+s"(kc), "+s"(vc), "+s"(kf), "+s"(vf), "+s"(qp));
    const int tmax = __builtin_amdgcn_readfirstlane(div_by(min(row0 + 31, M - 1), p.by_G));
    const int n_blocks = (L + tmax + 32) >> 5;                                // of 32 keys, visible to some row here
    const int n_my = w < n_blocks ? (n_blocks - w + kWaves - 1) / kWaves : 0;  // this wavefront's: w, w + 4, ..

    char* const mine = smem + w * kWaveLds;
    char* const q_lds = smem + kWaves * kWaveLds;
    const unsigned lds0 = (unsigned)(size_t)(lds_ptr)smem;
    const unsigned mine_lds = lds0 + w * kWaveLds;

    // ---- staging: one load instruction fills 4 rows of 256 B (1 KB): lane i -> row i >> 4, slot i & 15 ----
    const int lr = lane >> 4, ls = lane & 15;
    unsigned k_off[8], v_off[8];  // of this lane's piece in load u from a block's first row
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        k_off[u] = (unsigned)((4 * u + lr) * kv_row + ((ls ^ lr ^ ((u & 3) << 2)) << 4));
        v_off[u] = (unsigned)((4 * u + lr) * kv_row + ((ls ^ (lr << 1)) << 4));
    }
    auto stage = [&](int i) {  // block number i of this wavefront: K rows, then V rows (16 loads)
        const int j0 = (w + kWaves * i) * 32;
        const unsigned dst = mine_lds + (unsigned)(i & 1) * kStageBytes;
        const bool in_cache = j0 + 32 <= L;
        if (in_cache || (j0 >= L && j0 + 32 <= L + T)) {  // all rows from one tensor
            const int64_t from = (int64_t)(in_cache ? j0 : j0 - L) * kv_row + g * kRowBytes;
            // (both worked out and one taken: a choice between the pointers alone becomes one between their places in memory)
            const char *kb = kc + from, *vb = vc + from, *kb_run = kf + from, *vb_run = vf + from;
            asm volatile("" : "+s"(kb), "+s"(vb), "+s"(kb_run), "+s"(vb_run));
            load_lds16x8(in_cache ? kb : kb_run, k_off, dst);
            load_lds16x8(in_cache ? vb : vb_run, v_off, dst + kBlockBytes);
        } else {
            // Row j (rows past the last key repeat it: masked below) lies at base + j * kv_row, with one base for the cache's
            // rows and one for the run's: selects (written as a choice of expressions the compiler branches around every load).
#pragma unroll
            for (int is_v = 0; is_v < 2; ++is_v) {
                const unsigned long long in_c = (unsigned long long)((is_v ? vc : kc) + g * kRowBytes);
                const unsigned long long in_f = (unsigned long long)((is_v ? vf : kf) + g * kRowBytes) - (unsigned long long)L * (unsigned)kv_row;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const unsigned j = min(j0 + 4 * u + lr, L + T - 1);
                    const unsigned lo = (int)j < L ? (unsigned)in_c : (unsigned)in_f;
                    const unsigned up = (int)j < L ? (unsigned)(in_c >> 32) : (unsigned)(in_f >> 32);
                    const int piece = is_v ? ls ^ (lr << 1) : ls ^ lr ^ ((u & 3) << 2);
                    load_lds16(reinterpret_cast<const char*>(((unsigned long long)up << 32 | lo) + (unsigned long long)j * (unsigned)kv_row) + (piece << 4),
                               dst + is_v * kBlockBytes + u * 1024);
                }
            }
        }
    };
    // query rows: wavefront w brings rows 8 w .. 8 w + 7
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int r = 8 * w + 4 * u + lr, m = min(row0 + r, M - 1);
        const int t = div_by(m, p.by_G), hl = m - t * G;
        load_lds16(qp + ((int64_t)t * p.Hq + g * G + hl) * kRowBytes + ((ls ^ (r & 15)) << 4),
                   lds0 + kWaves * kWaveLds + (8 * w + 4 * u) * kRowBytes);
    }
    if (n_my > 0) stage(0);
    if (n_my > 1) stage(1);

    // this lane's query row and the last key it sees
    const int m_row = row0 + l32, t_row = div_by(min(m_row, M - 1), p.by_G);
    const int jmax = L + t_row;

    // the query rows are there for everybody (their two loads are the oldest of each wavefront's)
    if (n_my > 1) VS_WAIT_LOADS(32);
    else if (n_my > 0) VS_WAIT_LOADS(16);
    else VS_WAIT_LOADS(0);
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
    bf16x8 qf[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
        qf[kk] = *reinterpret_cast<const bf16x8*>(q_lds + l32 * kRowBytes + (((2 * kk + hi) ^ (l32 & 15)) << 4));

    int k_rd[8];  // K fragment kk: row l32, piece 2 kk + hi
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) k_rd[kk] = l32 * kRowBytes + (((2 * kk + hi) ^ (l32 & 15)) << 4);
    const int i16 = lane & 15, dh = (lane >> 4) & 1;
    int v_rd[2];  // V^T fragment corner, dim block parity x: row 4 hi + (i16 >> 2), piece 4 x + 2 dh + ((i16 & 3) >> 1)
#pragma unroll
    for (int x = 0; x < 2; ++x)
        v_rd[x] = (4 * hi + (i16 >> 2)) * kRowBytes + (((4 * x + 2 * dh + ((i16 & 3) >> 1)) ^ ((i16 >> 2) << 1)) << 4) + 8 * (i16 & 1);

    f32x16 o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    float m_ref = -INFINITY, l_run = 0.f;

    for (int i = 0; i < n_my; ++i) {
        const char* const kb = mine + (i & 1) * kStageBytes;
        const char* const vb = kb + kBlockBytes;
        const bool more = i + 1 < n_my;
        if (more) VS_WAIT_LOADS(24);  // K of this block has landed (behind it: its V and the next block)
        else VS_WAIT_LOADS(8);
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(kb + k_rd[kk]), qf[kk], s, 0, 0, 0);
        // lane (q = l32, hi), element e: key j0 + 8 (e >> 2) + 4 hi + (e & 3)
        const int j0 = (w + kWaves * i) * 32;
        float z[16];
        if (j0 + 32 > L) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                z[e] = j0 + 8 * (e >> 2) + 4 * hi + (e & 3) <= jmax ? s[e] * p.scale_log2e : -INFINITY;
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) z[e] = s[e] * p.scale_log2e;
        }
        float mx = z[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, z[e]);
        if (__any(mx > m_ref + kLazyMax)) {  // (always in the first block)
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_ref, mx);
            const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_ref - m_new);  // 0 while nothing is there
            m_ref = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
        }
        const float sub = m_ref == -INFINITY ? 0.f : m_ref;
        bf16x8 pf[2];
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            const bf16x2 pk = __builtin_convertvector(
                f32x2{__builtin_amdgcn_exp2f(z[e] - sub), __builtin_amdgcn_exp2f(z[e + 1] - sub)}, bf16x2);
            pf[e >> 3][e & 7] = pk[0];
            pf[e >> 3][(e & 7) + 1] = pk[1];
            l_run += (float)pk[0] + (float)pk[1];
        }
        if (more) VS_WAIT_LOADS(16);  // V of this block has landed
        else VS_WAIT_LOADS(0);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int db = 0; db < 4; ++db) {
                const char* const at = vb + v_rd[db & 1] + (db >> 1) * 128 + 16 * t * kRowBytes;
                const bf16x4 lo = lds_read_tr(at), hi4 = lds_read_tr(at + 8 * kRowBytes);
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7), pf[t], o[db], 0, 0, 0);
            }
        // the reads above are done (their values have been used): the stage is free for the block after next
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        if (i + 2 < n_my) stage(i + 2);
    }

    // ---- the four wavefronts meet in LDS: each leaves its sums in its own staging area, then closes dims 32 w .. 32 w + 31 ----
    float* const ml = reinterpret_cast<float*>(q_lds + kBlockBytes);  // [wavefront][row][2]
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (hi == 0) {
        ml[(w * 32 + l32) * 2] = m_ref;
        ml[(w * 32 + l32) * 2 + 1] = l_tot;
    }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
            *reinterpret_cast<f32x4*>(mine + ((db * 4 + e4) * 64 + lane) * 16) =
                f32x4{o[db][4 * e4], o[db][4 * e4 + 1], o[db][4 * e4 + 2], o[db][4 * e4 + 3]};
    __syncthreads();
    float mv[kWaves], lv[kWaves], m_star = -INFINITY, den = 0.f;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
        mv[v] = ml[(v * 32 + l32) * 2];
        lv[v] = ml[(v * 32 + l32) * 2 + 1];
        m_star = fmaxf(m_star, mv[v]);
    }
    f32x4 acc[4];
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) acc[e4] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
        const float a = mv[v] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mv[v] - m_star);
        den += a * lv[v];
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4)
            acc[e4] += a * *reinterpret_cast<const f32x4*>(smem + v * kWaveLds + ((w * 4 + e4) * 64 + lane) * 16);
    }
    // rows of the run that stay are copied into the cache, 16 bytes per thread, the workgroups of the launch
    // taking turns (no workgroup of this launch reads the cache rows written here)
    if (p.k_append_dst) {
        const int n16 = (T - p.append_first) * (kv_row / 16);
        const uint4* const ks = reinterpret_cast<const uint4*>(kf + (int64_t)p.append_first * kv_row);
        const uint4* const vs = reinterpret_cast<const uint4*>(vf + (int64_t)p.append_first * kv_row);
        for (int c = unit * kThreads + tid; c < n16; c += p.n_row_groups * p.Hkv * kThreads) {
            reinterpret_cast<uint4*>(p.k_append_dst)[c] = ks[c];
            reinterpret_cast<uint4*>(p.v_append_dst)[c] = vs[c];
        }
    }
    if (m_row >= M) return;
    const float inv = 1.0f / den;
    __bf16* const dst = p.out + ((int64_t)t_row * p.Hq + (int64_t)g * G + (m_row - t_row * G)) * D + 32 * w + 4 * hi;
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
        bf16x4 r;
#pragma unroll
        for (int j = 0; j < 4; ++j) r[j] = (__bf16)(acc[e4][j] * inv);
        *reinterpret_cast<bf16x4*>(dst + 8 * e4) = r;
    }
}

}  // namespace

hipError_t launch_prefill_short(const vs_shape& s, const void* kc, const void* vc, int32_t len, const void* q,
                                const void* kf, const void* vf, int32_t n_tokens, void* out, void* k_append_dst,
                                void* v_append_dst, hipStream_t st, bool append_all) {
    ShortParams p;
    p.kc = (const char*)kc;
    p.vc = (const char*)vc;
    p.q = (const char*)q;
    p.kf = (const char*)kf;
    p.vf = (const char*)vf;
    p.out = (__bf16*)out;
    p.k_append_dst = (char*)k_append_dst;
    p.v_append_dst = (char*)v_append_dst;
    p.append_first = append_all ? 0 : n_tokens - 1;
    p.L = len;
    p.T = n_tokens;
    p.G = s.n_q_heads / s.n_kv_heads;
    p.Hq = s.n_q_heads;
    p.Hkv = s.n_kv_heads;
    p.M = n_tokens * p.G;
    p.n_row_groups = (p.M + 31) / 32;
    p.units_per_xcd = (p.n_row_groups * p.Hkv + 7) / 8;
    p.scale_log2e = s.softmax_scale * kLog2e;
    p.by_G = quick_div(p.G);
    p.by_row_groups = quick_div(p.n_row_groups);
    static bool attr_set_on[16] = {};  // dynamic LDS above 64 KB has to be allowed once per kernel and device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return hipErrorInvalidDevice;
    if (!attr_set_on[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&prefill_short_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (e != hipSuccess) return e;
        attr_set_on[dev] = true;
    }
    prefill_short_kernel<<<8 * p.units_per_xcd, kThreads, kLds, st>>>(p);
    return hipGetLastError();
}

}  // namespace vs
