// The frame's rows and their Q/K/V projections for gfx950 (Section 3.1: Q = X W_Q, K = X W_K,
// V = X W_V; Section 3.3: the carrier's embedding is the mean of the frame's token embeddings;
// Section 3.2: it is the frame's last row).  One launch; X = [E ; mean(E)] is never written out,
// the outputs land in the layouts the frame prefill reads.
//
// N + 1 <= 192 rows meet n_out = (Hq + 2 Hkv) D weight rows of d numbers each.  A workgroup owns 32
// output features and all of the d input features, so nothing has to be added up across workgroups (there
// is no workspace to do it in).  64 input features at a time, a tile of the rows of E and 32 rows of W
// goes from global memory straight into LDS, whole 128-byte lines per 8 lanes, into a ring of tiles, the
// 16-byte pieces of a row stored permuted (piece ^ ((row >> 1) & 7)) so that the fragment reads of
// v_mfma_f32_16x16x32_bf16 (16 rows x one piece) hit all banks.  Four wavefronts multiply (wavefront w
// the 16-row sub-tiles w, w + 4, w + 8 with both 16-feature sub-tiles), four fetch; one barrier per tile.
//
// Every workgroup takes in all of E (1.2 MB with the weights' 0.2 at the 7B shape) through its compute
// unit, and that is what the launch is bound by: a request holds one of the 256 lines of the vector
// cache until its data is back and data comes back in order, so behind weights on their way from HBM the
// rows of E, which wait in L2, come in no faster than those: 28.9 us (51 GB/s per compute unit).  But 144
// workgroups leave 112 compute units idle: they run ahead as helpers and ask for the weight and embedding
// rows of the workgroups of their XCD, so that these find both in L2: 17.3 us over weights that the memory-side cache
// holds (30.9 without helpers, 23.6 with helpers for the weights alone, the same with 4 .. 16 loads of a helper's
// wavefront under way, 22.6 with 2), 17.6 .. 19.1 over 28 layers' weights.  When done the helpers sum up the carrier embedding.
//
// The carrier's row is not multiplied at all: the projection is linear, so its Q/K/V are the means
// over the token rows of the fp32 sums the workgroup holds anyway (the mean enters unrounded).
// The carrier embedding itself, if asked for, is computed on the side: each workgroup takes a
// share of the d columns and adds the rows in the order of mean_pool_kernel (16 row groups, then
// the groups in order, one division, one rounding), so it is the same bits as vs_carrier_mean_pool.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "vs_internal.h"

namespace vs {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kTileN = 32;       // output features per workgroup (2 sub-tiles of 16)
constexpr int kThreads = 512;
constexpr int kXcds = 8, kCus = 256;  // the chip the helpers are counted for: ids are dealt to the XCDs in turn
constexpr int kHelperDepth = 4;       // loads of a helper's wavefront under way: 8 x 4 KB fill the vector cache

struct QkvParams {
    const __bf16* e;   // [N][d]
    const __bf16* w;   // [n_out][d]
    __bf16* q;         // [N + 1][nq]
    __bf16* k;         // [N + 1][nk]
    __bf16* v;         // [N + 1][nk]
    __bf16* c_out;     // [d] or null
    int N, d, n_out, nq, nk;
    int n_blocks;      // workgroups that multiply; ids from n_blocks on are helpers
};

__device__ __forceinline__ __bf16* dest(const QkvParams& p, int m, int n) {
    if (n < p.nq) return p.q + (int64_t)m * p.nq + n;
    n -= p.nq;
    if (n < p.nk) return p.k + (int64_t)m * p.nk + n;
    return p.v + (int64_t)m * p.nk + (n - p.nk);
}

// The carrier embedding: share `part` of `parts` of the columns, by all threads of a workgroup.
__device__ __forceinline__ void pool_share(const QkvParams& p, int part, int parts, float (*poolsum)[32], int tid) {
    const int c_begin = (int)((int64_t)p.d * part / parts), c_end = (int)((int64_t)p.d * (part + 1) / parts);
    for (int c0 = c_begin; c0 < c_end; c0 += 32) {  // 32 columns x 16 row groups at a time
        const int col = c0 + (tid & 31), rg = tid >> 5;
        float sum = 0.f;
        if (col < c_end)
            for (int r = rg; r < p.N; r += 16) sum += (float)p.e[(int64_t)r * p.d + col];
        poolsum[rg][tid & 31] = sum;
        __syncthreads();
        if (tid < 32 && col < c_end) {
            float tot = poolsum[0][tid];
#pragma unroll
            for (int g = 1; g < 16; ++g) tot += poolsum[g][tid];
            p.c_out[col] = (__bf16)(tot / (float)p.N);
        }
        __syncthreads();
    }
}

template <int RS>
struct QkvTile {
    static constexpr int kRows = 64 * RS;  // rows of E a tile has room for
    static constexpr int kBytes = (kRows + kTileN) * 128;
    static constexpr int kRing = RS == 3 ? 5 : 6;
    static constexpr int kLds = kRing * kBytes;
};

// kNt: W is asked for as non-temporal and leaves the L2 to E, which pays where no helper has brought it there (192
// workgroups, 169 tokens, d 3584: 30.8 -> 28.5 us; 320, 1 token: 17.2 -> 15.8).
template <int RS, bool kNt>
__global__ __launch_bounds__(kThreads) void frame_qkv_kernel(QkvParams p) {
    using Tile = QkvTile<RS>;
    constexpr int kRows = Tile::kRows, kTileBytes = Tile::kBytes, kRing = Tile::kRing;
    extern __shared__ __attribute__((aligned(1024))) char ring[];  // kRing tiles: kRows rows of E, then 32 rows of W
    __shared__ float colsum[4][kTileN];
    __shared__ float poolsum[16][32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, kq = lane >> 4;
    const int N = p.N, d = p.d;
    const int n_tiles = d / 64;

    if ((int)blockIdx.x >= p.n_blocks) {
        // ---- a helper: the rows that the workgroups of this XCD (ids of the same residue) will ask for, tile by
        // tile, 8 rows (1 KB) per load, the wavefronts of the XCD's helpers taking turns ----
        const int x = blockIdx.x % kXcds;
        const int first = p.n_blocks + ((x - p.n_blocks) & (kXcds - 1));  // the XCD's first helper
        const int n_waves = (((int)gridDim.x - first + kXcds - 1) / kXcds) * 8;
        const int e_groups = (N + 7) / 8, w_groups = ((p.n_blocks - x + kXcds - 1) / kXcds) * (kTileN / 8);
        const int per_tile = e_groups + w_groups;
        int t = 0, u = (((int)blockIdx.x - first) / kXcds) * 8 + w;
        while (t < n_tiles) {
            u32x4 v[kHelperDepth];
#pragma unroll
            for (int k = 0; k < kHelperDepth; ++k) {
                while (u >= per_tile) {
                    u -= per_tile;
                    ++t;
                }
                const int r = lane >> 3;  // row of the group
                const __bf16* row;
                if (u < e_groups) {
                    row = p.e + (int64_t)min(u * 8 + r, N - 1) * d;
                } else {
                    const int g = u - e_groups, blk = x + kXcds * (g >> 2);
                    row = p.w + (int64_t)min(blk * kTileN + (g & 3) * 8 + r, p.n_out - 1) * d;
                }
                v[k] = *reinterpret_cast<const u32x4*>(row + (int64_t)min(t, n_tiles - 1) * 64 + (lane & 7) * 8);
                u += n_waves;
            }
#pragma unroll
            for (int k = 0; k < kHelperDepth; ++k) asm volatile("" : : "v"(v[k]));  // (nothing is done with them)
        }
        if (p.c_out) pool_share(p, blockIdx.x - p.n_blocks, gridDim.x - p.n_blocks, poolsum, tid);
        return;
    }

    const int n0 = blockIdx.x * kTileN;
    if (w >= 4) {
        // ---- global -> LDS.  A load instruction fills 8 rows: lane l -> row l >> 3, 16-byte slot l & 7,
        // which holds piece (l & 7) ^ ((row >> 1) & 7) of the row.  The four wavefronts take every
        // fourth group of 8 rows: those of E that exist, then the four of W.  (Written as assembly: for the builtin
        // form of these loads the compiler waits for all of them before any LDS read.  M0 is the LDS
        // address of the 1 KB; a write of M0 is kept one instruction away from its use.) ----
        const int e_groups = (N + 15) / 16 * 2, mine = (e_groups + kTileN / 8 - (w - 4) + 3) / 4;
        auto run = [&](auto n_loads) {
            constexpr int kLoads = decltype(n_loads)::value;
            unsigned off[kLoads], dst[kLoads];
            const char* base[kLoads];
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int grp = w - 4 + 4 * u, r8 = lane >> 3;
                const bool is_w = grp >= e_groups;
                const int r = (is_w ? grp - e_groups : grp) * 8 + r8;
                off[u] = (unsigned)(is_w ? min(r, p.n_out - 1 - n0) : min(r, N - 1)) * (unsigned)d * 2u +
                         (unsigned)(((lane & 7) ^ ((r >> 1) & 7)) << 4);
                dst[u] = (unsigned)(size_t)(lds_ptr)ring + (is_w ? kRows * 128 + (grp - e_groups) * 1024 : grp * 1024);
                base[u] = is_w ? reinterpret_cast<const char*>(p.w) + (int64_t)n0 * d * 2 : reinterpret_cast<const char*>(p.e);
            }
            auto issue = [&](int t, int slot) {
                if (t >= n_tiles) return;
#pragma unroll
                for (int u = 0; u < kLoads; ++u) {
                    if (kNt && u == kLoads - 1)  // (the four groups of W fall to the four wavefronts, last)
                        asm volatile("s_mov_b32 m0, %[dst]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o], %[b] nt"
                                     :
                                     : [dst] "s"(dst[u] + (unsigned)slot * kTileBytes), [o] "v"(off[u]), [b] "s"(base[u] + (int64_t)t * 128)
                                     : "memory");
                    else
                        asm volatile("s_mov_b32 m0, %[dst]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o], %[b]"
                                     :
                                     : [dst] "s"(dst[u] + (unsigned)slot * kTileBytes), [o] "v"(off[u]), [b] "s"(base[u] + (int64_t)t * 128)
                                     : "memory");
                }
            };
#pragma unroll
            for (int t = 0; t < kRing; ++t) issue(t, t);
            int slot = kRing - 1;
            for (int t = 0;; ++t) {
                // this wavefront's part of tile t has landed when no more than the tiles behind it are under way
                const int behind = min(t == 0 ? kRing - 1 : kRing - 2, n_tiles - 1 - t);
#pragma unroll
                for (int k = 0; k < kRing; ++k)
                    if (behind == k) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(k * kLoads) : "memory");
                __builtin_amdgcn_s_barrier();  // tile t is complete, and tile t-1 is in the registers of those who multiply
                if (t == n_tiles) break;
                if (t > 0) {
                    slot = slot + 1 == kRing ? 0 : slot + 1;
                    issue(t - 1 + kRing, slot);
                }
            }
        };
        using std::integral_constant;
        switch (mine) {
            case 1: run(integral_constant<int, 1>{}); break;
            case 2: run(integral_constant<int, 2>{}); break;
            case 3: run(integral_constant<int, 3>{}); break;
            case 4: run(integral_constant<int, 4>{}); break;
            case 5: run(integral_constant<int, 5>{}); break;
            case 6: run(integral_constant<int, 6>{}); break;
            default: run(integral_constant<int, 7>{}); break;  // (24 + 4 groups at most)
        }
    }

    f32x4 acc[RS][2];
#pragma unroll
    for (int i = 0; i < RS; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (w < 4) {
        // fragment reads: lane (i16, kq): piece h*4 + kq of row r for half h of the tile's 64 input features
        const int rd = i16 * 128 + ((kq ^ ((i16 >> 1) & 7)) << 4);  // ((row >> 1) & 7 is the same in every 16-row sub-tile)
        __builtin_amdgcn_s_barrier();  // tile 0 is complete
        asm volatile("" : : : "memory");
        bf16x8 af[2][2][RS], bfr[2][2][2];  // [register set][half][sub-tile]
        int slot = 0;
        auto read = [&](int set) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const char* const at = ring + ((slot * kTileBytes + rd) ^ (h * 64));
#pragma unroll
                for (int i = 0; i < RS; ++i) af[set][h][i] = *reinterpret_cast<const bf16x8*>(at + (w + 4 * i) * 2048);
#pragma unroll
                for (int ni = 0; ni < 2; ++ni) bfr[set][h][ni] = *reinterpret_cast<const bf16x8*>(at + kRows * 128 + ni * 2048);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto step = [&](int set) {
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // all of tile t is in registers
            __builtin_amdgcn_s_barrier();                          // so for everybody; and tile t+1 is complete
            asm volatile("" : : : "memory");
            slot = slot + 1 == kRing ? 0 : slot + 1;
            read(1 - set);  // tile t+1, while tile t is multiplied (behind the last one: whatever is there)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < RS; ++i)
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni)
                        acc[i][ni] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[set][h][i], bfr[set][h][ni], acc[i][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        read(0);
        for (int t = 0; t < n_tiles; t += 2) {
            step(0);
            if (t + 1 < n_tiles) step(1);
        }
    }
    __syncthreads();  // (the ring is free)

    // ---- the sums leave through LDS as a row-major tile, 8 neighbouring features of a row per thread.
    // lane (i16, kq) of acc[i][ni]: rows (w + 4 i)*16 + 4 kq + 0..3, feature n0 + 16 ni + i16.  Their column
    // sums make the carrier's row. ----
    float* const tile = reinterpret_cast<float*>(ring);  // [kRows][kTileN + 4]
    if (w < 4) {
        float csum[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < RS; ++i)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = (w + 4 * i) * 16 + 4 * kq + e;
                    if (m < N) csum[ni] += acc[i][ni][e];
                    tile[m * (kTileN + 4) + 16 * ni + i16] = acc[i][ni][e];
                }
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
            csum[ni] += __shfl_xor(csum[ni], 16);
            csum[ni] += __shfl_xor(csum[ni], 32);
            if (kq == 0) colsum[w][16 * ni + i16] = csum[ni];
        }
    }
    __syncthreads();
    if (tid < kTileN && n0 + tid < p.n_out)
        *dest(p, N, n0 + tid) =
            (__bf16)((((colsum[0][tid] + colsum[1][tid]) + colsum[2][tid]) + colsum[3][tid]) / (float)N);
    for (int idx = tid; idx < N * (kTileN / 8); idx += kThreads) {
        const int m = idx / (kTileN / 8), c8 = (idx % (kTileN / 8)) * 8;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(tile + m * (kTileN + 4) + c8);
        const f32x4 hi = *reinterpret_cast<const f32x4*>(tile + m * (kTileN + 4) + c8 + 4);
        const bf16x8 y = {(__bf16)lo[0], (__bf16)lo[1], (__bf16)lo[2], (__bf16)lo[3],
                          (__bf16)hi[0], (__bf16)hi[1], (__bf16)hi[2], (__bf16)hi[3]};
        // (head_dim is 128: a block of 32 features lies in one of the three tensors, and n_out is a multiple of it)
        *reinterpret_cast<bf16x8*>(dest(p, m, n0 + c8)) = y;
    }
    if (p.c_out && (int)gridDim.x == p.n_blocks) pool_share(p, blockIdx.x, gridDim.x, poolsum, tid);  // (no helpers)
}

// Helpers per XCD.  For a tile of 64 input features those of an XCD bring in `rows` rows (all of E, and W for the XCD's
// workgroups) at ~42 KB/us each; whoever multiplies takes (N + 32) rows at ~51 KB/us without their help, and no less than
// 0.22 us.  They pay while their time is below ~0.6 of that; slower ones only read everything a second time, and
// the launch waits for them (us with all idle compute units as helpers / with none, d 3584: 144 workgroups, 169 tokens 17.6 /
// 29.9, 1 token 11.9 / 12.3; 160: 24.6 / 30.5, 13.2 / 12.7; 180: 29.1 / 30.9, 13.8 / 12.8; 192: 32.6 / 30.8; 224: 52.9 /
// 31.5, 38.4 / 13.3; 240: 107.9 / 31.3).  The launch's fixed cost hides some more (192, d 1024: 10.4 / 11.9).  With a
// quarter of the multiplying workgroups' rows for each there are enough of them (24 workgroups, 169 tokens: 48 helpers
// 15.8, 232 helpers 15.7 us).  The counts are those of the whole chip: no helpers on a part of one.
int helpers_per_xcd(const QkvParams& p, int dev) {
    static int cus_of[16] = {};  // (asked for once per device)
    if (!cus_of[dev] && hipDeviceGetAttribute(&cus_of[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const int shift = xcd_shift_of_device(dev);  // (-1: not asked for yet)
    if (cus_of[dev] != kCus || (shift >= 0 && 1 << shift != kXcds)) return 0;
    const int idle = (kCus - p.n_blocks) / kXcds;
    if (idle < 2) return 0;
    const int rows = (p.N + 7) / 8 * 8 + kTileN * ((p.n_blocks + kXcds - 1) / kXcds), own = (p.N + 15) / 16 * 16 + kTileN;
    if (rows > idle * ((own > 84 ? own / 2 : 42) + 25600 / p.d)) return 0;
    const int enough = (4 * rows + own - 1) / own + 1;
    return enough < idle ? enough : idle;
}

}  // namespace

template <int RS, bool kNt>
hipError_t launch_qkv_variant(const QkvParams& p, int helpers, int dev, hipStream_t st) {
    static bool attr_set_on[16] = {};  // dynamic LDS above 64 KB has to be allowed once per kernel and device
    constexpr int kLds = QkvTile<RS>::kLds;
    if (!attr_set_on[dev]) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(&frame_qkv_kernel<RS, kNt>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (err != hipSuccess) return err;
        attr_set_on[dev] = true;
    }
    frame_qkv_kernel<RS, kNt><<<p.n_blocks + kXcds * helpers, kThreads, kLds, st>>>(p);
    return hipGetLastError();
}

template <int RS>
hipError_t launch_qkv_rows(const QkvParams& p, int dev, hipStream_t st) {
    const int helpers = helpers_per_xcd(p, dev);
    return helpers ? launch_qkv_variant<RS, false>(p, helpers, dev, st) : launch_qkv_variant<RS, true>(p, 0, dev, st);
}

hipError_t launch_frame_qkv(const vs_shape& s, const void* e, int32_t n_visual, int32_t d, const void* w,
                            void* q, void* k, void* v, void* c_out, hipStream_t st) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return hipErrorInvalidDevice;
    QkvParams p;
    p.e = (const __bf16*)e;
    p.w = (const __bf16*)w;
    p.q = (__bf16*)q;
    p.k = (__bf16*)k;
    p.v = (__bf16*)v;
    p.c_out = (__bf16*)c_out;
    p.N = n_visual;
    p.d = d;
    p.nq = s.n_q_heads * s.head_dim;
    p.nk = s.n_kv_heads * s.head_dim;
    p.n_out = p.nq + 2 * p.nk;
    p.n_blocks = (p.n_out + kTileN - 1) / kTileN;
    return n_visual <= 64 ? launch_qkv_rows<1>(p, dev, st)
                          : n_visual <= 128 ? launch_qkv_rows<2>(p, dev, st) : launch_qkv_rows<3>(p, dev, st);
}

}  // namespace vs
