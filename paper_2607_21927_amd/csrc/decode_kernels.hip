// Hybrid-Anchor decode step: the newest token of each sequence attends to the
// unique merge of its frozen stochastic anchor (the seed-ensemble union of the
// first generated position), its local window and the initial tokens, with
// one softmax per query head (Methods, "Hybrid Anchor and Pre-Fusion Unified
// Softmax").
//
// The key list of a (sequence, kv head) row is virtual and disjoint by
// construction: the anchor entries that fall neither in the window nor in the
// initial-token range, then the window [w_lo, t], then the initial tokens
// below the window.  Reading the three segments in turn is the unique()
// merge without sorting, and no index is visited twice.
//
// Split-K: the list is cut into 32-key tiles dealt round-robin to the P
// waves of the row (4 waves per workgroup), so any row length is covered
// whatever P the host picks.  A wave runs a flash-style pass over its tiles:
//   * S^T = K Q^T on MFMA 16x16x32 bf16, K rows gathered straight from HBM
//     into the A-operand layout (lane: key l%16, 8 dims at 8(l/16)), the G
//     query heads of the group as the 16-wide MFMA dimension;
//   * the online softmax per head (lane l owns head l%16; two cross-lane
//     exchanges per tile for the max);
//   * O += P V on MFMA with P packed to bf16 in registers and V staged
//     row-major in wave-private LDS and read transposed (ds_read_b64_tr_b16).
// The next tile's K/V loads issue before the current tile is computed.  K goes
// straight into the MFMA operand layout (64 bytes of a row per load); V, which
// passes through LDS anyway, is loaded as whole rows (187 against 190 us for
// 32 sequences at 64k, 16.7 against 18.4 us for one).  The four waves of a
// workgroup merge their states in LDS and write one partial (max, sum,
// unnormalised output) -- 1.6 instead of 6.3 MB of partials for one sequence
// at 64k, against 35 MB of K and V --; a second kernel merges the partials of
// each (sequence, query head).
#include "ris_device.h"
#include "ris_internal.h"

namespace ris {
namespace {

constexpr int kTileKeys = kDecodeTileKeys;
constexpr float kNegBig = -1e30f;   // finite start of the running max

struct RowSegs {
    int64_t na, nw, ns;   // anchor entries, window keys, initial keys below the window
    int64_t w_lo;         // window [w_lo, t]; initial tokens [0, ns)
    const int32_t* aidx;  // this row's anchor entries
};

// Key of virtual position v of the row, or -1 (an anchor entry already
// covered by the window or the initial range, or v past the end).
__device__ __forceinline__ int64_t key_of(const RowSegs& r, int64_t v) {
    if (v < r.na) {
        const int64_t j = r.aidx[v];
        return (j >= r.ns && j < r.w_lo) ? j : -1;
    }
    v -= r.na;
    if (v < r.nw) return r.w_lo + v;
    v -= r.nw;
    return v < r.ns ? v : -1;
}

template <int D>
struct KVTile {
    u32x4_t k[2][D / 32];
    u32x4_t v[2][D / 32];  // V rows, D / 8 lanes to a row: v[kb][s] is row 16 kb + (512 / D) s + lane / (D / 8)
    uint32_t valid;       // bit 16 kb + i: key slot 16 kb + i is a real key
};

template <int D, bool STREAM>
__device__ __forceinline__ void load_tile(const RowSegs& r, const uint16_t* Kr, const uint16_t* Vr,
                                          int64_t v0, int li, int lg, KVTile<D>& T) {
    uint32_t vm = 0;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int64_t j = key_of(r, v0 + 16 * kb + li);
        vm |= (uint32_t)(__ballot(j >= 0) & 0xFFFFull) << (16 * kb);
        const int64_t jj = j >= 0 ? j : 0;              // row 0 always exists
        const uint16_t* kp = Kr + jj * D + 8 * lg;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) T.k[kb][s] = *reinterpret_cast<const u32x4_t*>(kp + 32 * s);
        constexpr int LPR = D / 8, KPI = 64 / LPR;      // lanes per V row, V rows per load
        const int lane = li + 16 * lg;                  // max_len <= 2^31: a key fits 32 bits
#pragma unroll
        for (int s = 0; s < D / 32; ++s) {
            const int jv = __shfl((int)jj, KPI * s + lane / LPR);
            const u32x4_t* vp = reinterpret_cast<const u32x4_t*>(Vr + (int64_t)jv * D + 8 * (lane % LPR));
            T.v[kb][s] = STREAM ? __builtin_nontemporal_load(vp) : *vp;
        }
    }
    T.valid = vm;
}

__device__ __forceinline__ void store_out(const DecodeParams& p, int64_t at, float y) {
    if (p.out_bf16)
        static_cast<uint16_t*>(p.out)[at] = f32_to_bf16(y);
    else
        static_cast<float*>(p.out)[at] = y;
}

template <int D, bool STREAM>
__global__ __launch_bounds__(64 * kDecodeWaves, 2) void k_decode_partial(DecodeParams p, float c) {
    constexpr int SL = D / 32;         // k-slices of the score product
    constexpr int DB = D / 16;         // 16-dim blocks of the output
    constexpr int VS = D + 16;         // V row stride in LDS (bf16 elements)
    __shared__ __align__(16) uint16_t vlds[kDecodeWaves * kTileKeys * VS];
    __shared__ float2 ml[kDecodeWaves][8];   // the waves' (max, sum) per head
    static_assert(kTileKeys * VS * sizeof(uint16_t) >= 8 * D * sizeof(float), "a wave's outputs fit its V slice");

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int li = lane & 15, lg = lane >> 4;
    const int row = blockIdx.y;                       // b * Hkv + g
    const int b = row / p.Hkv, g = row - b * p.Hkv;
    const int G = p.G;
    const int64_t part = (int64_t)blockIdx.x * kDecodeWaves + wave;
    uint16_t* vw = vlds + wave * kTileKeys * VS;

    // ---- the row's three segments
    const int64_t t = p.pos[b];
    RowSegs r{0, 0, 0, 0, p.anchor_idx};
    if (t >= 0 && t < p.max_len) {
        const int64_t* ap = p.anchor_ptr + (int64_t)b * (p.Hkv + 1) + g;
        int64_t lo = ap[0], hi = ap[1];
        lo = lo < 0 ? 0 : (lo > p.anchor_stride ? p.anchor_stride : lo);
        hi = hi < lo ? lo : (hi > p.anchor_stride ? p.anchor_stride : hi);
        r.na = hi - lo;
        r.aidx = p.anchor_idx + (int64_t)b * p.anchor_stride + lo;
        r.w_lo = p.window > 0 ? (t - p.window + 1 > 0 ? t - p.window + 1 : 0) : t + 1;
        r.nw = t + 1 - r.w_lo;
        r.ns = p.sink < r.w_lo ? p.sink : r.w_lo;
    }
    const int64_t total = r.na + r.nw + r.ns;
    const int64_t stride = (int64_t)p.parts * kTileKeys;   // this wave's tiles: part, part + P, ...
    const uint16_t* Kr = static_cast<const uint16_t*>(p.K) + (int64_t)row * p.max_len * D;
    const uint16_t* Vr = static_cast<const uint16_t*>(p.V) + (int64_t)row * p.max_len * D;

    // ---- Q^T as the B operand: lane l holds head l%16, dims 32 s + 8 (l/16) ..
    u32x4_t qf[SL];
    {
        const bool hv = li < G;
        const uint16_t* qp = static_cast<const uint16_t*>(p.Q) +
                             ((int64_t)b * p.Hq + (int64_t)g * G + (hv ? li : 0)) * D + 8 * lg;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const u32x4_t v = *reinterpret_cast<const u32x4_t*>(qp + 32 * s);
            qf[s] = hv ? v : zero;
        }
    }

    f32x4_t o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float m_run = kNegBig, l_run = 0.f;

    const int64_t v_first = part * kTileKeys;
    if (v_first < total) {
        KVTile<D> cur;
        load_tile<D, STREAM>(r, Kr, Vr, v_first, li, lg, cur);
        for (int64_t v0 = v_first; v0 < total; v0 += stride) {
            KVTile<D> nxt;
            const bool more = v0 + stride < total;
            if (more) load_tile<D, STREAM>(r, Kr, Vr, v0 + stride, li, lg, nxt);

            // V rows into this wave's LDS, row-major.
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int s = 0; s < SL; ++s)
                    *reinterpret_cast<u32x4_t*>(vw + (16 * kb + (512 / D) * s + lane / (D / 8)) * VS + 8 * (lane % (D / 8))) = cur.v[kb][s];

            // S^T = K Q^T: lane l holds head l%16 at key slots 16 kb + 4 (l/16) + i.
            f32x4_t st[2];
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                st[kb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < SL; ++s)
                    st[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(cur.k[kb][s]),
                                                                      as_bf16x8(qf[s]), st[kb], 0, 0, 0);
            }

            // Online softmax over the tile (scores in the log2 domain).
            float sc[2][4];
            float mx = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bool ok = (cur.valid >> (16 * kb + 4 * lg + i)) & 1u;
                    sc[kb][i] = ok ? st[kb][i] * c : -INFINITY;
                    mx = fmaxf(mx, sc[kb][i]);
                }
            mx = quad_max16(mx);
            const float m_new = fmaxf(m_run, mx);
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            float pv[2][4];
            float ps = 0.f;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    pv[kb][i] = __builtin_amdgcn_exp2f(sc[kb][i] - m_new);
                    ps += pv[kb][i];
                }
            l_run = l_run * alpha + ps;
            m_run = m_new;

            // Rescale the output rows: lane l holds heads 4 (l/16) + i.
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float a = __shfl(alpha, 4 * lg + i);
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db][i] *= a;
            }

            // P as the A operand: head l%16, k slots 8 (l/16) + e hold keys
            // 4 (l/16) + e (e < 4) and 16 + 4 (l/16) + e - 4 (e >= 4).
            const u32x4_t pk = {pack_bf16x2(pv[0][0], pv[0][1]), pack_bf16x2(pv[0][2], pv[0][3]),
                                pack_bf16x2(pv[1][0], pv[1][1]), pack_bf16x2(pv[1][2], pv[1][3])};
            // V as the B operand with the same key order: lane l addresses key
            // row l/4 (then 16 + l/4) at dims 16 db + 4 (l%4).
            const uint16_t* v_lo = vw + (lane >> 2) * VS + 4 * (lane & 3);
            const uint16_t* v_hi = v_lo + 16 * VS;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint2 a = lds_read_tr16(v_lo + 16 * db);
                const uint2 e = lds_read_tr16(v_hi + 16 * db);
                const u32x4_t vb = {a.x, a.y, e.x, e.y};
                o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(pk), as_bf16x8(vb), o[db], 0, 0, 0);
            }
            if (more) cur = nxt;
        }
    }

    // ---- the workgroup's partial: the four waves' states merged in LDS (each
    // wave's V slice is free once its own last tile is done, but the merge's
    // rows span other waves' slices, hence the first barrier)
    l_run = quad_sum16(l_run);
    __syncthreads();
    float* ow = reinterpret_cast<float*>(vlds);             // [wave][head][dim]
    if (lane < G) ml[wave][lane] = make_float2(m_run, l_run);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int h = 4 * lg + i;
        if (h < G) {
#pragma unroll
            for (int db = 0; db < DB; ++db) ow[(wave * G + h) * D + 16 * db + li] = o[db][i];
        }
    }
    __syncthreads();
    const int64_t slot = (int64_t)row * gridDim.x + blockIdx.x;
    float* pml = p.part_ml + slot * G * 2;
    float* po = p.part_o + slot * G * D;
    for (int e = threadIdx.x; e < G * D; e += 64 * kDecodeWaves) {
        const int h = e / D;
        float M = ml[0][h].x;
#pragma unroll
        for (int w = 1; w < kDecodeWaves; ++w) M = fmaxf(M, ml[w][h].x);
        float O = 0.f, L = 0.f;
#pragma unroll
        for (int w = 0; w < kDecodeWaves; ++w) {
            const float c = __builtin_amdgcn_exp2f(ml[w][h].x - M);
            O += c * ow[w * G * D + e];
            L += c * ml[w][h].y;
        }
        if (gridDim.x == 1) {                                // the row's only partial: its output
            store_out(p, (int64_t)row * G * D + e, L > 0.f ? (O + 0.f) / L : 0.f);
            continue;
        }
        po[e] = O;
        if (e % D == 0) {
            pml[2 * h] = M;
            pml[2 * h + 1] = L;
        }
    }
}

// Merge the workgroups' partials of one (sequence, query head): the threads first find the
// common max and each partial's weight together (in LDS); then D/4 lanes of
// four dims each sum over every kGroups-th partial, and the groups' sums meet
// in LDS.  Latency-bound (a batch of one has 256 partials of 512 bytes a head):
// one thread per dim walking every partial took 48 us there.
constexpr int kCombineThreads = 256;
template <int D>
__global__ __launch_bounds__(kCombineThreads) void k_decode_combine(DecodeParams p, int parts) {
    constexpr int kLanes = D / 4, kGroups = kCombineThreads / kLanes;
    __shared__ float wgt[kDecodeMaxParts / kDecodeWaves];
    __shared__ float red[kCombineThreads / 64][2];
    __shared__ __align__(16) float osum[kGroups][D];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t bh = blockIdx.x;
    const int b = (int)(bh / p.Hq), h = (int)(bh % p.Hq);
    const int g = h / p.G, hh = h - g * p.G;
    const int64_t row = (int64_t)b * p.Hkv + g;
    const int64_t step_ml = p.G, step_o = (int64_t)p.G * D;
    const float2* ml = reinterpret_cast<const float2*>(p.part_ml) + row * parts * step_ml + hh;
    const float* po = p.part_o + row * parts * step_o + (int64_t)hh * D;
    float M = kNegBig;
    for (int i = tid; i < parts; i += kCombineThreads) M = fmaxf(M, ml[i * step_ml].x);
    M = wave_max(M);
    if (lane == 0) red[wv][0] = M;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kCombineThreads / 64; ++w) M = fmaxf(M, red[w][0]);
    float L = 0.f;
    for (int i = tid; i < parts; i += kCombineThreads) {
        const float2 x = ml[i * step_ml];
        const float w = __builtin_amdgcn_exp2f(x.x - M);
        wgt[i] = w;
        L += w * x.y;
    }
    L = wave_sum(L);
    if (lane == 0) red[wv][1] = L;
    __syncthreads();
    const int grp = tid / kLanes, d4 = 4 * (tid % kLanes);
    f32x4_t O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int i = grp; i < parts; i += kGroups) O += wgt[i] * *reinterpret_cast<const f32x4_t*>(po + i * step_o + d4);
    *reinterpret_cast<f32x4_t*>(&osum[grp][d4]) = O;
    __syncthreads();
    if (tid < D) {
        L = 0.f;
#pragma unroll
        for (int w = 0; w < kCombineThreads / 64; ++w) L += red[w][1];
        float y = 0.f;
#pragma unroll
        for (int k = 0; k < kGroups; ++k) y += osum[k][tid];
        y = L > 0.f ? y / L : 0.f;
        const int64_t at = bh * D + tid;
        store_out(p, at, y);
    }
}

// K and V bytes of a step from which V is read past the caches (non-temporal
// loads of whole rows; K's 64-byte pieces need the cache for a row's other
// pieces).  The bytes are an estimate from the descriptor, and an upper one: an
// anchor's capacity counts every draw, and window and initial tokens may lie in it
// (70 seeds at 1% of 64k, window 1,024: 48 MB a sequence for 33 MB read).
// Measured in the caches / past them, 12/2 heads of 128, each step with the caches
// full of other data, as between a model's layers: 4 sequences (192 MB by the
// estimate) 135 / 129 us with the fill, 5 (240) 156 / 146, 6 (288) 166 / 156, 8
// (384) 175 / 160, 12 (575) 232 / 221; the same step over and over: 31.0 / 31.4,
// 44.2 / 46.0, 51.6 / 51.9, 50.6 / 50.6, 108 / 92, 32 sequences 201 / 182.  32/4 heads
// of 64, over and over: 5 sequences 34.2 / 37.3, 6 40.3 / 43.2, 7 47.9 / 48.9, 8
// 54.6 / 53.1, 12 92 / 78; with other data 147 / 138, 158 / 148, 169 / 156, 174 / 160,
// 212 / 200.  The line lies where the repeated step loses little any more.
constexpr int64_t kStreamBytes = 256ll << 20;

template <int D>
hipError_t launch_d(const DecodeParams& p, float c, hipStream_t st) {
    const dim3 grid((unsigned)(p.parts / kDecodeWaves), (unsigned)(p.B * p.Hkv));
    if (p.parts % kDecodeWaves != 0 || p.parts > kDecodeMaxParts) return hipErrorInvalidValue;
    if (p.kv_bytes > kStreamBytes)
        hipLaunchKernelGGL((k_decode_partial<D, true>), grid, dim3(64 * kDecodeWaves), 0, st, p, c);
    else
        hipLaunchKernelGGL((k_decode_partial<D, false>), grid, dim3(64 * kDecodeWaves), 0, st, p, c);
    hipError_t e = hipGetLastError();
    // One partial a row is the row's output.  (Short rows: 8/8 heads of 64, 110 keys,
    // one sequence 6.6 us with one thread per dim merging four partials, 6.9 with
    // the merge above and this launch, 4.3 without.)
    if (e != hipSuccess || grid.x == 1) return e;
    hipLaunchKernelGGL(k_decode_combine<D>, dim3((unsigned)((int64_t)p.B * p.Hq)), dim3(kCombineThreads), 0, st, p,
                       p.parts / kDecodeWaves);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_decode(const DecodeParams& p, hipStream_t st) {
    const float c = p.scale * 1.4426950408889634f;   // scores in the log2 domain
    return p.D == 128 ? launch_d<128>(p, c, st) : launch_d<64>(p, c, st);
}

}  // namespace ris
