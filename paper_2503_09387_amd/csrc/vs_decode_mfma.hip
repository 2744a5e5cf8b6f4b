// Decode attention for bf16 storage on gfx950 (VideoScan Section 3.3, decoding phase;
// Eq. 1 of Section 3.1): one query token per stream over that stream's retained rows.
//
// The step is bound by reading K and V once from HBM, so the work is cut by ROWS, not by
// stream: the 32-row tiles of all streams are laid end to end and every workgroup of the
// launch takes an equal, contiguous share of them (a share that crosses from one stream into
// the next is worked off as two segments).  A workgroup reads WHOLE rows: its wavefronts are
// the KV heads (wavefront w walks the share for head w), so together they stream contiguous
// memory, which HBM serves measurably faster than one head's 256 bytes out of every 1 KB.
// (With fewer than 4 KV heads the spare wavefronts take sub-ranges of the share; with more,
// blockIdx.y selects the group of 4 heads.)  The grid is one workgroup per compute unit, so
// they all run at once and stream for the whole launch.  A wavefront works alone, with no
// barrier anywhere in the kernel:
//   * K and V rows are loaded coalesced and parked row-major in wave-private LDS buffers; K comes
//     back as the A operand of v_mfma_f32_16x16x32_bf16 (S^T = K Q^T; the G query heads of the KV
//     head are the columns, padded to 16), V transposed through ds_read_b64_tr_b16 for
//     O^T += V^T P^T.  (Loaded straight in the operand's layout, 16 rows of 64 bytes per
//     instruction, a K tile kept the compute unit's load path four times as long: 8 tiles in one
//     workgroup 8.1 -> 6.8 us, one stream of 512 rows over 16 workgroups 9.4 -> 9.25 us with its
//     merge; no difference at 16 long streams.)
//   * the next tile's 16 KB are already in flight while the current tile is computed;
//   * the softmax reference maximum is refreshed only when a score exceeds it by more than
//     2^8, which needs one ballot per tile instead of two cross-lane reductions and one
//     accumulator rescale.
// The row appended in this step is read from k_new / v_new (never from the slab, which the
// wavefront that owns the stream's last tile updates on the side).  Every wavefront leaves a
// normalised partial result (fp16 with a power-of-two scale per row) with its reference and sum; a second small kernel merges
// them (a launch that follows another on the same stream starts within about a microsecond of
// it; what the merge costs is its one round trip to memory).  For few rows there is a kernel
// that merges inside the launch, further down.
#include "vs_internal.h"

namespace vs {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int D = 128;
constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int TR = 32;      // rows per wave tile
constexpr int VSTR = 144;   // LDS row stride of the V tile in elements (288 B)
constexpr int KSTR = 136;   // and of the K tile (272 B)
constexpr int kWaveLds = TR * (VSTR + KSTR) * 2;  // bytes: V tile, then K tile
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLazyMax = 8.0f;  // scores may exceed the reference maximum by 2^8 before it is refreshed

struct DecodeParams {
    __bf16* k_slab;
    __bf16* v_slab;
    const __bf16* q;
    const __bf16* k_new;  // may be null
    const __bf16* v_new;
    __bf16* out;
    // partial results: [slot][Hkv][nsub][G][D] normalised, slot = workgroup + stream of the segment; stored
    // as fp16 after multiplying the row by the power of two that brings its largest entry into
    // [2^14, 2^15) (11 significant bits whatever the size of the values, in the bytes of bf16)
    _Float16* part_o;
    float* part_ml;       // [slot][Hkv][nsub][G][4]: reference (log2 units), sum, inverse of the row's scale, unused
    int64_t stream_stride;   // elements between streams in the slabs
    int n_streams, G, Hq, Hkv;
    int nh, nsub;            // KV heads per workgroup (1, 2 or 4) and sub-ranges per share (4 / nh)
    int n_wg;                // workgroups along x
    int total_tiles;         // tile_prefix[n_streams]
    int share_q, share_r;    // total_tiles = n_wg * share_q + share_r: the first share_r workgroups take share_q + 1 tiles
    float scale_log2e;
    LenTable lens;           // valid rows per stream, the appended row included
    int tile_prefix[kMaxStreamsPerLaunch + 1];  // tiles of the streams before this one
    int first_wg[kMaxStreamsPerLaunch];  // first workgroup (along x) that holds tiles of the stream, and how many do:
    int n_wgs[kMaxStreamsPerLaunch];     // what the merge kernel walks
};

// first flat tile of workgroup w (w = n_wg gives the end)
__device__ __forceinline__ int wg_first_tile(const DecodeParams& p, int w) {
    return w * p.share_q + min(w, p.share_r);
}

__device__ __forceinline__ bf16x4 lds_read_tr(const __bf16* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
        (__attribute__((address_space(3))) bf16x4*)(p));
}

// One tile (32 rows) of one wave: scores, lazy-reference softmax, value accumulation.
// The K and V tiles have been parked in the wave's LDS buffers.
#define VS_KFRAG(HALF, SLICE) (*reinterpret_cast<const bf16x8*>(krd + 16 * (HALF) * KSTR + 32 * (SLICE)))
#define VS_TILE_COMPUTE(R0)                                                                           \
    do {                                                                                              \
        f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = sa;                                                     \
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(0, 0), qf0, sa, 0, 0, 0);               \
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(1, 0), qf0, sb, 0, 0, 0);               \
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(0, 1), qf1, sa, 0, 0, 0);               \
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(1, 1), qf1, sb, 0, 0, 0);               \
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(0, 2), qf2, sa, 0, 0, 0);               \
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(1, 2), qf2, sb, 0, 0, 0);               \
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(0, 3), qf3, sa, 0, 0, 0);               \
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(VS_KFRAG(1, 3), qf3, sb, 0, 0, 0);               \
        float z[8];                                                                                   \
        _Pragma("unroll") for (int e = 0; e < 4; ++e) {                                               \
            z[e] = ((R0) + 4 * kq + e < row_end) ? sa[e] * p.scale_log2e : -INFINITY;                 \
            z[4 + e] = ((R0) + 16 + 4 * kq + e < row_end) ? sb[e] * p.scale_log2e : -INFINITY;        \
        }                                                                                             \
        float mx = fmaxf(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])),                                 \
                         fmaxf(fmaxf(z[4], z[5]), fmaxf(z[6], z[7])));                                \
        if (__any(mx > m_ref + kLazyMax)) { /* rare after the first tile: refresh the reference */    \
            mx = fmaxf(mx, __shfl_xor(mx, 16));                                                       \
            mx = fmaxf(mx, __shfl_xor(mx, 32));                                                       \
            const float m_new = fmaxf(m_ref, mx); /* finite: the tile has a valid row */              \
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new); /* 0 on the first tile */      \
            m_ref = m_new;                                                                            \
            l_run *= alpha;                                                                           \
            o0 *= alpha; o1 *= alpha; o2 *= alpha; o3 *= alpha;                                       \
            o4 *= alpha; o5 *= alpha; o6 *= alpha; o7 *= alpha;                                       \
        }                                                                                             \
        bf16x8 pf;                                                                                    \
        _Pragma("unroll") for (int e = 0; e < 8; ++e) {                                               \
            const float pe = __builtin_amdgcn_exp2f(z[e] - m_ref);                                    \
            l_run += pe;                                                                              \
            pf[e] = (__bf16)pe;                                                                       \
        }                                                                                             \
        VS_PV(o0, 0); VS_PV(o1, 1); VS_PV(o2, 2); VS_PV(o3, 3);                                       \
        VS_PV(o4, 4); VS_PV(o5, 5); VS_PV(o6, 6); VS_PV(o7, 7);                                       \
    } while (0)

#define VS_PV(ACC, DB)                                                                          \
    do {                                                                                        \
        const bf16x4 lo = lds_read_tr(vrd + 16 * (DB));                                         \
        const bf16x4 hi4 = lds_read_tr(vrd + 16 * VSTR + 16 * (DB));                            \
        ACC = __builtin_amdgcn_mfma_f32_16x16x32_bf16(                                          \
            __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7), pf, ACC, 0, 0, 0);        \
    } while (0)

#define VS_KPTR(row) (((row) == new_row ? knew : kslab + (int64_t)(row) * row_stride) + 8 * i16)
#define VS_VPTR(row) (((row) == new_row ? vnew : vslab + (int64_t)(row) * row_stride) + 8 * i16)
// every K/V byte is read once by one wavefront: the loads are marked non-temporal
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_nt(const void* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
}
#define VS_LD(ptr) ld_nt(ptr)
// loads one tile into the register set named by suffix X: 8 K and 8 V row pieces (individually named
// registers, so that nothing lands in scratch)
#define VS_FETCH(tile, X)                                                            \
    do {                                                                             \
        const int fr0 = row_begin + (tile) * TR;                                     \
        k0##X = VS_LD(VS_KPTR(min(fr0 + kq, last)));                                 \
        k1##X = VS_LD(VS_KPTR(min(fr0 + 4 + kq, last)));                            \
        k2##X = VS_LD(VS_KPTR(min(fr0 + 8 + kq, last)));                            \
        k3##X = VS_LD(VS_KPTR(min(fr0 + 12 + kq, last)));                           \
        k4##X = VS_LD(VS_KPTR(min(fr0 + 16 + kq, last)));                           \
        k5##X = VS_LD(VS_KPTR(min(fr0 + 20 + kq, last)));                           \
        k6##X = VS_LD(VS_KPTR(min(fr0 + 24 + kq, last)));                           \
        k7##X = VS_LD(VS_KPTR(min(fr0 + 28 + kq, last)));                           \
        v0##X = VS_LD(VS_VPTR(min(fr0 + kq, last)));                                 \
        v1##X = VS_LD(VS_VPTR(min(fr0 + 4 + kq, last)));                             \
        v2##X = VS_LD(VS_VPTR(min(fr0 + 8 + kq, last)));                             \
        v3##X = VS_LD(VS_VPTR(min(fr0 + 12 + kq, last)));                            \
        v4##X = VS_LD(VS_VPTR(min(fr0 + 16 + kq, last)));                            \
        v5##X = VS_LD(VS_VPTR(min(fr0 + 20 + kq, last)));                            \
        v6##X = VS_LD(VS_VPTR(min(fr0 + 24 + kq, last)));                            \
        v7##X = VS_LD(VS_VPTR(min(fr0 + 28 + kq, last)));                            \
    } while (0)
#define VS_PARK_ROW(n, kreg, vreg)                                                   \
    do {                                                                             \
        *reinterpret_cast<uint4*>(&vs_k[(4 * (n) + kq) * KSTR + 8 * i16]) = kreg;     \
        *reinterpret_cast<uint4*>(&vs_w[(4 * (n) + kq) * VSTR + 8 * i16]) = vreg;     \
    } while (0)
#define VS_PARK(X)                                                                   \
    do {                                                                             \
        VS_PARK_ROW(0, k0##X, v0##X); VS_PARK_ROW(1, k1##X, v1##X);                  \
        VS_PARK_ROW(2, k2##X, v2##X); VS_PARK_ROW(3, k3##X, v3##X);                  \
        VS_PARK_ROW(4, k4##X, v4##X); VS_PARK_ROW(5, k5##X, v5##X);                  \
        VS_PARK_ROW(6, k6##X, v6##X); VS_PARK_ROW(7, k7##X, v7##X);                  \
    } while (0)

// Grid (n_wg, Hkv / nh).
__global__ __launch_bounds__(kThreads, 2) void decode_mfma_kernel(DecodeParams p) {
    __shared__ __attribute__((aligned(16))) char smem[kWaves * kWaveLds];  // per-wave V and K tiles

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, kq = lane >> 4;
    const int g = blockIdx.y * p.nh + wave % p.nh;  // this wavefront's KV head
    const int sub = wave / p.nh;                     // and its sub-range of every segment
    const int64_t row_stride = (int64_t)p.Hkv * D;
    const int flat_end = wg_first_tile(p, blockIdx.x + 1);
    int flat = wg_first_tile(p, blockIdx.x);
    // Lane i holds the end of stream i in flat tiles and its length: one fetch at the start, and
    // whatever a segment needs of a stream is then read out of these registers (a fetch per
    // segment would sit between the workgroup's start and its first K/V loads).
    static_assert(kMaxStreamsPerLaunch <= 64, "one lane per stream");
    const int end_of = p.tile_prefix[min(lane, kMaxStreamsPerLaunch - 1) + 1];
    const int len_of = p.lens.v[min(lane, kMaxStreamsPerLaunch - 1)];
    // stream of the first tile: the number of streams that end at or before it
    int s = __builtin_popcountll(__ballot(end_of <= flat));
    __bf16* vs_w = reinterpret_cast<__bf16*>(smem + wave * kWaveLds);
    __bf16* vs_k = vs_w + TR * VSTR;
    const __bf16* krd = &vs_k[i16 * KSTR + 8 * kq];
    const __bf16* vrd = &vs_w[(4 * kq + (i16 >> 2)) * VSTR + 4 * (i16 & 3)];

  for (; flat < flat_end; ++s) {
    // ---- one segment: tiles [seg_a, seg_b) of stream s; this wavefront takes the sub-range
    //      [tile_a, tile_b) of it for head g ----
    const int len = __builtin_amdgcn_readlane(len_of, s);
    const int first_of = s ? __builtin_amdgcn_readlane(end_of, s - 1) : 0;
    const int stream_tiles = __builtin_amdgcn_readlane(end_of, s) - first_of;
    const int seg_a = flat - first_of;
    const int seg_b = min(stream_tiles, flat_end - first_of);
    const bool whole_stream = seg_a == 0 && seg_b == stream_tiles && p.nsub == 1;
    const int tile_a = seg_a + (seg_b - seg_a) * sub / p.nsub;
    const int tile_b = seg_a + (seg_b - seg_a) * (sub + 1) / p.nsub;
    const int row_begin = tile_a * TR;
    const int row_end = min(len, tile_b * TR);
    const int n_tiles = tile_b - tile_a;
    const int last = max(row_end - 1, 0);
    const int new_row = p.k_new ? len - 1 : -1;
    __bf16* kslab = p.k_slab + (int64_t)s * p.stream_stride + (int64_t)g * D;
    __bf16* vslab = p.v_slab + (int64_t)s * p.stream_stride + (int64_t)g * D;
    const __bf16* knew = p.k_new ? p.k_new + ((int64_t)s * p.Hkv + g) * D : nullptr;
    const __bf16* vnew = p.v_new ? p.v_new + ((int64_t)s * p.Hkv + g) * D : nullptr;

    // two tiles are requested before anything else happens
    const uint4 zz = make_uint4(0, 0, 0, 0);
    uint4 k0a = zz, k1a = zz, k2a = zz, k3a = zz, k4a = zz, k5a = zz, k6a = zz, k7a = zz;
    uint4 v0a = zz, v1a = zz, v2a = zz, v3a = zz, v4a = zz, v5a = zz, v6a = zz, v7a = zz;
    uint4 k0b = zz, k1b = zz, k2b = zz, k3b = zz, k4b = zz, k5b = zz, k6b = zz, k7b = zz;
    uint4 v0b = zz, v1b = zz, v2b = zz, v3b = zz, v4b = zz, v5b = zz, v6b = zz, v7b = zz;
    if (0 < n_tiles) VS_FETCH(0, a);
    if (1 < n_tiles) VS_FETCH(1, b);

    // the step's new row also goes into the slab (nobody reads it from there in this launch):
    // done by the wavefront whose range ends with the stream's last tile
    if (new_row >= 0 && n_tiles > 0 && tile_b == stream_tiles && lane < 32) {
        const int c = lane & 15;
        const uint4* src = reinterpret_cast<const uint4*>(lane < 16 ? knew : vnew) + c;
        uint4* dst = reinterpret_cast<uint4*>((lane < 16 ? kslab : vslab) + (int64_t)new_row * row_stride) + c;
        *dst = *src;
    }

    // Q^T fragments (B operand): lane (col = i16, k = 8*kq..8*kq+7), zero beyond the G heads
    bf16x8 qf0, qf1, qf2, qf3;
    {
        const __bf16* qrow = p.q + ((int64_t)s * p.Hq + (int64_t)g * p.G + min(i16, p.G - 1)) * D + 8 * kq;
        const unsigned int keep = i16 < p.G ? 0xffffffffu : 0u;
        uint4 a = VS_LD(qrow), b = VS_LD(qrow + 32), c = VS_LD(qrow + 64), d = VS_LD(qrow + 96);
        a.x &= keep; a.y &= keep; a.z &= keep; a.w &= keep;
        b.x &= keep; b.y &= keep; b.z &= keep; b.w &= keep;
        c.x &= keep; c.y &= keep; c.z &= keep; c.w &= keep;
        d.x &= keep; d.y &= keep; d.z &= keep; d.w &= keep;
        qf0 = __builtin_bit_cast(bf16x8, a);
        qf1 = __builtin_bit_cast(bf16x8, b);
        qf2 = __builtin_bit_cast(bf16x8, c);
        qf3 = __builtin_bit_cast(bf16x8, d);
    }

    f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0, o2 = o0, o3 = o0, o4 = o0, o5 = o0, o6 = o0, o7 = o0;
    float m_ref = -INFINITY, l_run = 0.f;  // m_ref: softmax reference (log2 units), uniform per head column

    // the LDS buffer is private to the wave, whose LDS operations execute in program order
    for (int t = 0; t < n_tiles; t += 2) {
        VS_PARK(a);
        VS_TILE_COMPUTE(row_begin + t * TR);
        if (t + 2 < n_tiles) VS_FETCH(t + 2, a);
        if (t + 1 < n_tiles) {
            VS_PARK(b);
            VS_TILE_COMPUTE(row_begin + (t + 1) * TR);
            if (t + 3 < n_tiles) VS_FETCH(t + 3, b);
        }
    }

    // ---- this wavefront's result: lane (head = i16, kq) holds dims 16*db + 4*kq + e ----
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    {
        const float inv = l_run > 0.f ? 1.0f / l_run : 0.f;
        const int head = min(i16, p.G - 1);  // (lanes beyond the G heads compute along and store nothing)
        if (whole_stream) {
            __bf16* dst = p.out + ((int64_t)s * p.Hq + (int64_t)g * p.G + head) * D + 4 * kq;
#define VS_OUT(ACC, DB)                                                                  \
            do {                                                                         \
                bf16x4 r_;                                                               \
                _Pragma("unroll") for (int j = 0; j < 4; ++j) r_[j] = (__bf16)(ACC[j] * inv); \
                if (i16 < p.G) *reinterpret_cast<bf16x4*>(dst + 16 * (DB)) = r_;         \
            } while (0)
            VS_OUT(o0, 0); VS_OUT(o1, 1); VS_OUT(o2, 2); VS_OUT(o3, 3);
            VS_OUT(o4, 4); VS_OUT(o5, 5); VS_OUT(o6, 6); VS_OUT(o7, 7);
#undef VS_OUT
        } else {
            // the row's largest entry: this lane holds 32 of its dims, lanes +-16, +-32 the rest
            float big = 0.f;
#define VS_BIG(ACC) big = fmaxf(fmaxf(fmaxf(big, fabsf(ACC[0])), fmaxf(fabsf(ACC[1]), fabsf(ACC[2]))), fabsf(ACC[3]))
            VS_BIG(o0); VS_BIG(o1); VS_BIG(o2); VS_BIG(o3); VS_BIG(o4); VS_BIG(o5); VS_BIG(o6); VS_BIG(o7);
#undef VS_BIG
            big *= inv;
            big = fmaxf(big, __shfl_xor(big, 16));
            big = fmaxf(big, __shfl_xor(big, 32));
            const int expo = (int)((__float_as_uint(big) >> 23) & 255u);
            const int se = min(max(127 + 14 + 127 - expo, 1), 254);  // biased exponent of the scale
            const float scale = __uint_as_float((unsigned)se << 23), inv_scale = __uint_as_float((unsigned)(254 - se) << 23);
            const int64_t pr = ((((int64_t)blockIdx.x + s) * p.Hkv + g) * p.nsub + sub) * p.G + head;
            _Float16* dst = p.part_o + pr * D + 4 * kq;
            if (kq == 0 && i16 < p.G) *reinterpret_cast<float4*>(p.part_ml + pr * 4) = make_float4(m_ref, l_run, inv_scale, 0.f);
#define VS_OUT(ACC, DB)                                                                  \
            do {                                                                         \
                f16x4 r_;                                                                \
                _Pragma("unroll") for (int j = 0; j < 4; ++j) r_[j] = (_Float16)((ACC[j] * inv) * scale); \
                if (i16 < p.G) *reinterpret_cast<f16x4*>(dst + 16 * (DB)) = r_;          \
            } while (0)
            VS_OUT(o0, 0); VS_OUT(o1, 1); VS_OUT(o2, 2); VS_OUT(o3, 3);
            VS_OUT(o4, 4); VS_OUT(o5, 5); VS_OUT(o6, 6); VS_OUT(o7, 7);
#undef VS_OUT
        }
    }
    flat = first_of + seg_b;  // next segment: the next stream
  }
}
// ---- few rows: one launch, merged inside ----
// With few rows a step is a chain of latencies, and the second launch with its trip to memory is
// 3 us of 8.  Here a workgroup is a share of ONE stream's rows for one KV head: its W wavefronts
// take sub-ranges of the share (a tile or two each) and meet in LDS.  A stream of several shares
// then passes fp32 partial results (G rows of 512 bytes per share) through memory at agent scope:
// stores and loads that pass the L2s, which are not coherent with each other; every store
// acknowledged before the workgroup counts itself in; the last one to arrive adds the shares in
// index order, and nobody waits.  The counter goes back to where it started with the last arrival.
// The upper 24 bits of a counter are a mark that vs_workspace_init puts there.  In memory that has been used for
// something else since (or was never prepared) they are something else; every arrival sees that,
// whatever the order, and the stream's first share then does the whole stream by itself: right, but slower (one stream
// of 700 / 3000 rows 15.4 / 30.1 us).
// A caller without a workspace (counters null) keeps no state between launches: the shares are then
// added by decode_shares_kernel, a launch of its own, in the same order and so to the same bits.
// Measured (28/4 heads, us per call, this kernel and the two launches): 1 stream of 128 rows 5.3 / 7.8,
// of 256 6.8 / 7.7, of 700 8.6 / 8.8; 16 streams of 700 10.9 / 12.5, of 3000 22.7 / 25.5; 64 of 700 20.0 / 24.8.
struct ShortParams {
    __bf16* k_slab;
    __bf16* v_slab;
    const __bf16* q;
    const __bf16* k_new;  // may be null
    const __bf16* v_new;
    __bf16* out;
    float* part_o;        // [share][Hkv][G][D], not normalised
    float* part_ml;       // [share][Hkv][G][2]: reference (log2 units), sum
    unsigned* counters;   // [stream][Hkv], kDecodeCounterStart between launches; null: the shares are added by a second launch
    int64_t stream_stride;
    int G, Hq, Hkv;
    float scale_log2e;
    LenTable lens;        // valid rows per stream, the appended row included
    int share_end[kMaxStreamsPerLaunch];  // shares of the streams up to and with this one
};

__device__ __forceinline__ void store_agent(float* dst, float a, float b) {
    const unsigned long long v = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(dst), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_agent(const float* src) {
    const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(src), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
    return make_float2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}

// The shares of stream s, KV head g, added in index order: dims dp, dp + 1 of query head `head` of the group.  kAgent: the partial
// results were stored in this launch, by other workgroups.
template <bool kAgent>
__device__ __forceinline__ void add_shares(const ShortParams& p, int s, int g, int first_share, int n_shares, int head, int dp) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    constexpr int kDepth = 8;
    const int64_t pr0 = ((int64_t)first_share * p.Hkv + g) * p.G + head, step = (int64_t)p.Hkv * p.G;
    float mref = -INFINITY, l = 0.f, a = 0.f, b = 0.f;
    for (int j0 = 0; j0 < n_shares; j0 += kDepth) {
        float2 ml[kDepth], o[kDepth];
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const int64_t pr = pr0 + min(j0 + u, n_shares - 1) * step;
            ml[u] = kAgent ? load_agent(p.part_ml + pr * 2) : *reinterpret_cast<const float2*>(p.part_ml + pr * 2);
            o[u] = kAgent ? load_agent(p.part_o + pr * D + dp) : *reinterpret_cast<const float2*>(p.part_o + pr * D + dp);
        }
        float mx = mref;
#pragma unroll
        for (int u = 0; u < kDepth; ++u) mx = fmaxf(mx, ml[u].x);
        const float f = __builtin_amdgcn_exp2f(mref - mx);  // 0 before the first batch
        l *= f;
        a *= f;
        b *= f;
        mref = mx;
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const float w = j0 + u < n_shares ? __builtin_amdgcn_exp2f(ml[u].x - mx) : 0.f;
            l += w * ml[u].y;
            a += w * o[u].x;
            b += w * o[u].y;
        }
    }
    const float inv = 1.0f / l;
    *reinterpret_cast<bf16x2*>(p.out + ((int64_t)s * p.Hq + (int64_t)g * p.G + head) * D + dp) =
        bf16x2{(__bf16)(a * inv), (__bf16)(b * inv)};
}

// Grid (shares of all streams, Hkv).
template <int W>
__global__ __launch_bounds__(64 * W, 2) void decode_short_kernel(ShortParams p) {
    constexpr int kRowStride = D + 4;                                        // of a head's sums in LDS, in floats
    constexpr int kWaveBytes = kWaveLds;
    static_assert(kMaxGroup * kRowStride * 4 <= kWaveBytes, "a wavefront's sums take the place of its V tile");
    __shared__ __attribute__((aligned(16))) char smem[W * kWaveBytes];
    __shared__ float s_m[W][16], s_l[W][16];
    __shared__ unsigned s_before;

  // once; a second time only where the first share of a stream does the whole stream
  for (bool alone = false;; alone = true) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, kq = lane >> 4;
    const int g = blockIdx.y, share = blockIdx.x;
    const int64_t row_stride = (int64_t)p.Hkv * D;
    static_assert(kMaxStreamsPerLaunch == 64, "one lane per stream");
    const int end_of = p.share_end[lane];
    const int len_of = p.lens.v[lane];
    const int s = __builtin_popcountll(__ballot(end_of <= share));
    const int len = __builtin_amdgcn_readlane(len_of, s);
    const int first_share = s ? __builtin_amdgcn_readlane(end_of, s - 1) : 0;
    const int n_shares = alone ? 1 : __builtin_amdgcn_readlane(end_of, s) - first_share, j_share = share - first_share;
    const int stream_tiles = (len + TR - 1) / TR;
    const int new_row = p.k_new ? len - 1 : -1;
    __bf16* kslab = p.k_slab + (int64_t)s * p.stream_stride + (int64_t)g * D;
    __bf16* vslab = p.v_slab + (int64_t)s * p.stream_stride + (int64_t)g * D;
    const __bf16* knew = p.k_new ? p.k_new + ((int64_t)s * p.Hkv + g) * D : nullptr;
    const __bf16* vnew = p.v_new ? p.v_new + ((int64_t)s * p.Hkv + g) * D : nullptr;
    __bf16* vs_w = reinterpret_cast<__bf16*>(smem + wave * kWaveBytes);
    __bf16* vs_k = vs_w + TR * VSTR;
    const __bf16* krd = &vs_k[i16 * KSTR + 8 * kq];
    const __bf16* vrd = &vs_w[(4 * kq + (i16 >> 2)) * VSTR + 4 * (i16 & 3)];
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const int n_items = p.G * (D / 2);  // (head, pair of dims)
    const int seg_a = stream_tiles * j_share / n_shares, seg_b = stream_tiles * (j_share + 1) / n_shares;
    const int tile_a = seg_a + (seg_b - seg_a) * wave / W;
    const int tile_b = seg_a + (seg_b - seg_a) * (wave + 1) / W;
    const int row_begin = tile_a * TR;
    const int row_end = min(len, tile_b * TR);
    const int n_tiles = tile_b - tile_a;
    const int last = max(row_end - 1, 0);
    f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0, o2 = o0, o3 = o0, o4 = o0, o5 = o0, o6 = o0, o7 = o0;
    float m_ref = -INFINITY, l_run = 0.f;
    if (n_tiles > 0) {
        const uint4 zz = make_uint4(0, 0, 0, 0);
        uint4 k0a, k1a, k2a, k3a, k4a, k5a, k6a, k7a, v0a, v1a, v2a, v3a, v4a, v5a, v6a, v7a;
        uint4 k0b = zz, k1b = zz, k2b = zz, k3b = zz, k4b = zz, k5b = zz, k6b = zz, k7b = zz;
        uint4 v0b = zz, v1b = zz, v2b = zz, v3b = zz, v4b = zz, v5b = zz, v6b = zz, v7b = zz;
        VS_FETCH(0, a);
        if (1 < n_tiles) VS_FETCH(1, b);
        if (new_row >= 0 && tile_b == stream_tiles && lane < 32) {  // (nobody reads the slab's copy in this launch)
            const int c = lane & 15;
            const uint4* src = reinterpret_cast<const uint4*>(lane < 16 ? knew : vnew) + c;
            uint4* dst = reinterpret_cast<uint4*>((lane < 16 ? kslab : vslab) + (int64_t)new_row * row_stride) + c;
            *dst = *src;
        }
        bf16x8 qf0, qf1, qf2, qf3;
        {
            const __bf16* qrow = p.q + ((int64_t)s * p.Hq + (int64_t)g * p.G + min(i16, p.G - 1)) * D + 8 * kq;
            const uint4 a = VS_LD(qrow), b = VS_LD(qrow + 32), c = VS_LD(qrow + 64), d = VS_LD(qrow + 96);
            qf0 = __builtin_bit_cast(bf16x8, a);  // (columns beyond the G heads repeat the last one and are not used)
            qf1 = __builtin_bit_cast(bf16x8, b);
            qf2 = __builtin_bit_cast(bf16x8, c);
            qf3 = __builtin_bit_cast(bf16x8, d);
        }
        for (int t = 0; t < n_tiles; t += 2) {
            VS_PARK(a);
            VS_TILE_COMPUTE(row_begin + t * TR);
            if (t + 2 < n_tiles) VS_FETCH(t + 2, a);
            if (t + 1 < n_tiles) {
                VS_PARK(b);
                VS_TILE_COMPUTE(row_begin + (t + 1) * TR);
                if (t + 3 < n_tiles) VS_FETCH(t + 3, b);
            }
        }
        l_run += __shfl_xor(l_run, 16);
        l_run += __shfl_xor(l_run, 32);
    }

    // ---- the wavefronts meet in LDS ----
    if (kq == 0) {
        s_m[wave][i16] = m_ref;
        s_l[wave][i16] = l_run;
    }
    __syncthreads();
    {
        float mx = s_m[0][i16];
#pragma unroll
        for (int w = 1; w < W; ++w) mx = fmaxf(mx, s_m[w][i16]);
        const float f = __builtin_amdgcn_exp2f(m_ref - mx);  // 0 for a wavefront without rows
        float* row = reinterpret_cast<float*>(smem + wave * kWaveBytes) + i16 * kRowStride + 4 * kq;
        if (i16 < p.G) {
#define VS_OUT(ACC, DB) *reinterpret_cast<f32x4*>(row + 16 * (DB)) = ACC * f
            VS_OUT(o0, 0); VS_OUT(o1, 1); VS_OUT(o2, 2); VS_OUT(o3, 3);
            VS_OUT(o4, 4); VS_OUT(o5, 5); VS_OUT(o6, 6); VS_OUT(o7, 7);
#undef VS_OUT
        }
    }
    __syncthreads();
    for (int it = tid; it < n_items; it += 64 * W) {
        const int head = it / (D / 2), dp = 2 * (it % (D / 2));
        float mx = s_m[0][head];
#pragma unroll
        for (int w = 1; w < W; ++w) mx = fmaxf(mx, s_m[w][head]);
        float l = 0.f, a = 0.f, b = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            l += s_l[w][head] * __builtin_amdgcn_exp2f(s_m[w][head] - mx);
            const float2 v = *reinterpret_cast<const float2*>(reinterpret_cast<const float*>(smem + w * kWaveBytes) + head * kRowStride + dp);
            a += v.x;
            b += v.y;
        }
        if (n_shares == 1) {
            const float inv = 1.0f / l;
            *reinterpret_cast<bf16x2*>(p.out + ((int64_t)s * p.Hq + (int64_t)g * p.G + head) * D + dp) =
                bf16x2{(__bf16)(a * inv), (__bf16)(b * inv)};
        } else {
            const int64_t pr = ((int64_t)share * p.Hkv + g) * p.G + head;
            store_agent(p.part_o + pr * D + dp, a, b);
            if (dp == 0) store_agent(p.part_ml + pr * 2, mx, l);
        }
    }
    if (n_shares == 1 || !p.counters) return;

    // ---- the shares of the stream: the last to arrive adds them ----
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's partial results have arrived
    __syncthreads();
    unsigned* const counter = p.counters + s * p.Hkv + g;
    if (tid == 0) s_before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const unsigned before = __builtin_amdgcn_readfirstlane(s_before);
    if ((before & kDecodeCounterMark) != kDecodeCounterStart) {  // not prepared, or overwritten
        if (j_share == 0) continue;
        return;
    }
    if (before - kDecodeCounterStart != (unsigned)(n_shares - 1)) return;
    if (tid == 0) __hip_atomic_store(counter, kDecodeCounterStart, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int it = tid; it < n_items; it += 64 * W) add_shares<true>(p, s, g, first_share, n_shares, it / (D / 2), 2 * (it % (D / 2)));
    return;
  }
}

// The shares of a stream added by a launch of their own.  Grid (streams, Hq), a wavefront each.
__global__ __launch_bounds__(64) void decode_shares_kernel(ShortParams p) {
    const int s = blockIdx.x, first_share = s ? p.share_end[s - 1] : 0, n_shares = p.share_end[s] - first_share;
    const int g = blockIdx.y / p.G;
    if (n_shares > 1) add_shares<false>(p, s, g, first_share, n_shares, blockIdx.y - g * p.G, 2 * threadIdx.x);
}
#undef VS_TILE_COMPUTE
#undef VS_PV
#undef VS_KPTR
#undef VS_VPTR
#undef VS_LD
#undef VS_FETCH
#undef VS_PARK
#undef VS_PARK_ROW
#undef VS_KFRAG

// Merge of a stream's partials (a stream that one wavefront per head covered alone was written
// directly).  Grid (streams, query heads), one wavefront each = 4 groups of 16 lanes: a lane owns
// 8 output dims and the partials group, group + 4, ..; up to kDepth of them per lane are
// requested at once (one round trip to memory for up to 64 partials), merged in the lane in index
// order, and the four groups are then merged with two lane exchanges.  No LDS, no barrier.  A depth that
// fits the number of partials leaves out loads that only repeat the last one: one stream of 700 rows
// 9.45 -> 8.8 us per call; four wavefronts for more than 64: one stream of 8192 rows 17.2 -> 13.1 us.
// kDepth: partials a group requests at once.  kCW > 1 (streams of more than 64 partials): that many
// wavefronts, the groups of all of them dealing the partials out, which then meet in LDS.
constexpr int kCombineGroups = 4;
template <int kDepth, int kCW>
__global__ __launch_bounds__(64 * kCW) void decode_combine_kernel(DecodeParams p) {
    const int s = blockIdx.x, hq = blockIdx.y;
    const int w_first = p.first_wg[s], n_wgs = p.n_wgs[s];
    if (n_wgs == 1 && p.nsub == 1) return;
    const int g = hq / p.G, h = hq - g * p.G;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, pg = lane >> 4, t = lane & 15, d8 = t * 8;
    const int n_parts = n_wgs * p.nsub;
    // partial c of the stream: workgroup w_first + c / nsub, sub-range c % nsub
    const int64_t slot_rows = (int64_t)p.Hkv * p.nsub * p.G;
    auto row_of = [&](int c) {
        const int w = p.nsub == 1 ? c : c / p.nsub, sub = p.nsub == 1 ? 0 : c - w * p.nsub;
        return ((int64_t)(w_first + w + s) * slot_rows) + ((int64_t)g * p.nsub + sub) * p.G + h;
    };
    float acc[8], den = 0.f, mref = -INFINITY;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    constexpr int kStep = kCombineGroups * kCW;
    for (int c0 = wave * kCombineGroups + pg; c0 < n_parts; c0 += kStep * kDepth) {
        float4 ml[kDepth];  // reference, sum, inverse scale of the stored row
        f16x8 o[kDepth];
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const int c = min(c0 + kStep * u, n_parts - 1);  // (past the end: a valid row, ignored below)
            const int64_t pr = row_of(c);
            ml[u] = *reinterpret_cast<const float4*>(p.part_ml + pr * 4);
            o[u] = *reinterpret_cast<const f16x8*>(p.part_o + pr * D + d8);
        }
#pragma unroll
        for (int u = 0; u < kDepth; ++u)
            if (c0 + kStep * u >= n_parts) ml[u] = make_float4(-INFINITY, 0.f, 0.f, 0.f);
        float mx = mref;
#pragma unroll
        for (int u = 0; u < kDepth; ++u) mx = fmaxf(mx, ml[u].x);
        if (mx == -INFINITY) continue;
        const float sc = (mref == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mref - mx);
        den *= sc;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= sc;
        mref = mx;
#pragma unroll
        for (int u = 0; u < kDepth; ++u) {
            const float wt = (ml[u].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ml[u].x - mx) * ml[u].y;
            den += wt;
            const float wo = wt * ml[u].z;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] += wo * (float)o[u][j];
        }
    }
    // the four groups: (0, 1) and (2, 3) first, then the pairs
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
        const float m2 = __shfl_xor(mref, off), d2 = __shfl_xor(den, off);
        const float mx = fmaxf(mref, m2);
        const float a0 = (mref == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mref - mx);
        const float a1 = (m2 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m2 - mx);
        // (both lanes of a pair must add in the same order to end up with the same bits: the lower group first)
        const bool low = (lane & off) == 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float x2 = __shfl_xor(acc[j], off);
            acc[j] = low ? acc[j] * a0 + x2 * a1 : x2 * a1 + acc[j] * a0;
        }
        den = low ? den * a0 + d2 * a1 : d2 * a1 + den * a0;
        mref = mx;
    }
    if constexpr (kCW > 1) {
        __shared__ float s_acc[kCW][16][9], s_m[kCW], s_d[kCW];  // (9: rows of 8 apart from one another in the banks)
        if (pg == 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) s_acc[wave][t][j] = acc[j];
            if (t == 0) {
                s_m[wave] = mref;
                s_d[wave] = den;
            }
        }
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int w = 1; w < kCW; ++w) {
            const float m2 = s_m[w], mx = fmaxf(mref, m2);
            const float a0 = (mref == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mref - mx);
            const float a1 = (m2 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m2 - mx);
            den = den * a0 + s_d[w] * a1;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = acc[j] * a0 + s_acc[w][t][j] * a1;
            mref = mx;
        }
    }
    if (pg != 0) return;
    const float inv = 1.0f / den;
    bf16x8 r;
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = (__bf16)(acc[j] * inv);
    *reinterpret_cast<bf16x8*>(p.out + ((int64_t)s * p.Hq + hq) * D + d8) = r;
}

constexpr int kDecodeMaxWorkgroups = 1024;

// KV heads per workgroup (one wavefront each): the largest of 1, 2, 4 that divides Hkv; the
// other wavefronts take sub-ranges of the share.  One rule for the sizing and the launch.
int heads_per_workgroup(int n_kv_heads) { return n_kv_heads % 4 == 0 ? 4 : (n_kv_heads % 2 == 0 ? 2 : 1); }

// Whether a step is one of few rows, and its shares: wavefronts per workgroup (0: the kernel that shares
// all rows out equally) and tiles per share.
struct ShortPlan {
    int waves, tiles;
};
inline int shares_of(int rows, int tiles) { return ((rows + TR - 1) / TR + tiles - 1) / tiles; }

// All workgroups must run at once, one per compute unit.  Measured at 28/4, 16/2, 24/8 and 12/6 heads, 1 to 64
// streams of 64 to 8192 rows (us per call, this kernel / the two launches):
//   * up to 8 tiles per stream: one share each and no merge, 4 wavefronts up to 4 tiles;
//   * up to 32 tiles: shares of 4 tiles (8.6 / 8.8 at 1 x 700, 9.2 / 9.5 at 4 x 700; shares of 8: 9.0, 9.6);
//   * beyond, the fewest tiles from 8 on with which the shares fit the chip, up to 24 (23.2 / 25.5 at 8 x 6000;
//     32 tiles, 8 x 8192: 30.4 / 29.5) and up to 12 shares per stream, which one workgroup adds
//     (24 and 32 shares, 1 x 6000 and 1 x 8192: 12.4 / 11.9 and 13.7 / 13.1);
//   * shares are cut per stream: where ragged streams would leave the largest share more than 1.4 times
//     its equal part of the rows, the other kernel's equal shares are better, except at 8 tiles, where
//     latency decides and not the amount (10.4 / 11.0 at 4 x 1500).
ShortPlan short_plan(const LenTable& lens, int n_streams, int n_kv_heads) {
    int64_t total = 0;
    int most = 0;
    for (int i = 0; i < n_streams; ++i) {
        const int t = (lens.v[i] + TR - 1) / TR;
        total += t;
        most = t > most ? t : most;
    }
    constexpr int kChip = 256, kMaxTiles = 24, kMaxShares = 12;
    auto fits = [&](int tiles) {
        int64_t n = 0;
        for (int i = 0; i < n_streams; ++i) n += shares_of(lens.v[i], tiles);
        return n * n_kv_heads <= kChip;
    };
    if (most > kMaxTiles * kMaxShares || total * n_kv_heads > (int64_t)kChip * kMaxTiles) return {0, 0};
    if (most <= 4 && fits(4)) return {4, 4};
    if (most > 8 && most <= 32 && fits(4)) return {4, 4};
    for (int tiles = 8; tiles <= kMaxTiles; ++tiles) {
        if ((most + tiles - 1) / tiles > kMaxShares || !fits(tiles)) continue;
        if (tiles > 8 && 5.0 * tiles * kChip > 7.0 * (double)total * n_kv_heads) break;
        return {8, tiles};
    }
    return {0, 0};
}

// Rows of partial results: a slot per (workgroup + stream of the segment), each with one row per
// (KV head, sub-range, query head of the group).
int64_t partial_rows(const vs_shape& s, int32_t n_streams) {
    const int G = s.n_q_heads / s.n_kv_heads, nsub = kWaves / heads_per_workgroup(s.n_kv_heads);
    return ((int64_t)kDecodeMaxWorkgroups + n_streams) * s.n_kv_heads * nsub * G;
}

}  // namespace

size_t decode_mfma_workspace_bytes(const vs_shape& s, int32_t n_streams, int32_t /*max_rows*/) {
    return (size_t)(partial_rows(s, n_streams) * (D * sizeof(_Float16) + 4 * sizeof(float)));
}

hipError_t launch_decode_mfma(const vs_shape& s, int32_t n_streams, void* k_slab, void* v_slab,
                              int32_t capacity, const LenTable& lens, const void* q,
                              const void* k_new, const void* v_new, void* out, void* counters,
                              void* workspace, hipStream_t st) {
    const ShortPlan plan = g_tune_decode_chunk_rows ? ShortPlan{0, 0} : short_plan(lens, n_streams, s.n_kv_heads);
    if (plan.waves) {
        ShortParams h;
        h.k_slab = (__bf16*)k_slab;
        h.v_slab = (__bf16*)v_slab;
        h.q = (const __bf16*)q;
        h.k_new = (const __bf16*)k_new;
        h.v_new = (const __bf16*)v_new;
        h.out = (__bf16*)out;
        h.stream_stride = (int64_t)capacity * s.n_kv_heads * D;
        h.G = s.n_q_heads / s.n_kv_heads;
        h.Hq = s.n_q_heads;
        h.Hkv = s.n_kv_heads;
        h.scale_log2e = s.softmax_scale * kLog2e;
        h.lens = lens;
        int n = 0;
        for (int i = 0; i < kMaxStreamsPerLaunch; ++i) {
            if (i < n_streams) n += shares_of(lens.v[i], plan.tiles);
            h.share_end[i] = i < n_streams ? n : 0x7fffffff;  // (never "before" a share)
        }
        // (at most 256 shares of 520 bytes per query head; the workspace holds more than 1024 x 272)
        h.counters = (unsigned*)counters;
        h.part_ml = (float*)workspace;
        h.part_o = h.part_ml + (int64_t)n * s.n_q_heads * 2;
        const dim3 grid(n, s.n_kv_heads);
        if (plan.waves == 4) decode_short_kernel<4><<<grid, 256, 0, st>>>(h);
        else decode_short_kernel<8><<<grid, 512, 0, st>>>(h);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || counters || n == n_streams) return e;  // (n == n_streams: one share each)
        decode_shares_kernel<<<dim3(n_streams, s.n_q_heads), 64, 0, st>>>(h);
        return hipGetLastError();
    }
    DecodeParams p;
    p.k_slab = (__bf16*)k_slab;
    p.v_slab = (__bf16*)v_slab;
    p.q = (const __bf16*)q;
    p.k_new = (const __bf16*)k_new;
    p.v_new = (const __bf16*)v_new;
    p.out = (__bf16*)out;
    p.stream_stride = (int64_t)capacity * s.n_kv_heads * D;
    p.n_streams = n_streams;
    p.G = s.n_q_heads / s.n_kv_heads;
    p.Hq = s.n_q_heads;
    p.Hkv = s.n_kv_heads;
    p.nh = heads_per_workgroup(s.n_kv_heads);
    p.nsub = kWaves / p.nh;
    p.scale_log2e = s.softmax_scale * kLog2e;
    p.lens = lens;
    p.tile_prefix[0] = 0;
    for (int i = 0; i < n_streams; ++i) p.tile_prefix[i + 1] = p.tile_prefix[i] + (lens.v[i] + TR - 1) / TR;
    for (int i = n_streams; i < kMaxStreamsPerLaunch; ++i) p.tile_prefix[i + 1] = 0x7fffffff;  // never "before" a tile
    p.total_tiles = p.tile_prefix[n_streams];
    // Shares of equal size in tiles, one workgroup per compute unit (measured on cfg4: 256 workgroups
    // 30.0 us, 512 30.7 us, and anything in between worse, because some compute units then hold two
    // workgroups and the others one; fewer shares also mean fewer partial results to merge); the
    // tuning knob gives the rows per share instead.
    const int groups_y = s.n_kv_heads / p.nh;
    const int max_x = groups_y < 256 ? 256 / groups_y : 1;
    int64_t tiles_per_wg = g_tune_decode_chunk_rows ? g_tune_decode_chunk_rows / TR : (p.total_tiles + max_x - 1) / max_x;
    if (tiles_per_wg < p.nsub) tiles_per_wg = p.nsub;
    int64_t n_wg = (p.total_tiles + tiles_per_wg - 1) / tiles_per_wg;
    if (n_wg > kDecodeMaxWorkgroups) n_wg = kDecodeMaxWorkgroups;
    if (n_wg < 1) n_wg = 1;
    p.n_wg = (int)n_wg;
    p.share_q = p.total_tiles / p.n_wg;
    p.share_r = p.total_tiles % p.n_wg;
    // which workgroups hold a stream: the largest w with first tile <= the stream's first / last tile
    {
        const int big = p.share_r * (p.share_q + 1);  // tiles held by the workgroups with one tile more
        auto owner = [&](int tile) {
            return tile < big ? tile / (p.share_q + 1) : p.share_r + (tile - big) / (p.share_q > 0 ? p.share_q : 1);
        };
        for (int i = 0; i < kMaxStreamsPerLaunch; ++i) {
            p.first_wg[i] = 0;
            p.n_wgs[i] = 1;
            if (i < n_streams && p.tile_prefix[i + 1] > p.tile_prefix[i]) {
                p.first_wg[i] = owner(p.tile_prefix[i]);
                p.n_wgs[i] = owner(p.tile_prefix[i + 1] - 1) - p.first_wg[i] + 1;
            }
        }
    }
    // the largest slot a wavefront can name is (n_wg - 1) + (n_streams - 1)
    const int64_t rows = partial_rows(s, n_streams);
    if ((int64_t)(p.n_wg + n_streams - 1) * s.n_kv_heads * p.nsub * p.G > rows) return hipErrorInvalidValue;
    p.part_ml = (float*)workspace;
    p.part_o = (_Float16*)(p.part_ml + rows * 4);
    const dim3 grid(p.n_wg, groups_y);
    decode_mfma_kernel<<<grid, kThreads, 0, st>>>(p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int most = 1;  // partials of a stream
    for (int i = 0; i < n_streams; ++i) most = p.n_wgs[i] * p.nsub > most ? p.n_wgs[i] * p.nsub : most;
    const dim3 cgrid(n_streams, s.n_q_heads);
    if (most <= 4 * kCombineGroups) decode_combine_kernel<4, 1><<<cgrid, 64, 0, st>>>(p);
    else if (most <= 8 * kCombineGroups) decode_combine_kernel<8, 1><<<cgrid, 64, 0, st>>>(p);
    else if (most <= 16 * kCombineGroups) decode_combine_kernel<16, 1><<<cgrid, 64, 0, st>>>(p);
    else decode_combine_kernel<16, 4><<<cgrid, 256, 0, st>>>(p);
    return hipGetLastError();
}

}  // namespace vs
