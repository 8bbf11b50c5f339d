// Elementwise layers of the host models around the sparse attention: the
// residual add fused with RMSNorm, and the SwiGLU activation of the MLP.
// Both are HBM-bound; one pass over the data each, float32 arithmetic.
#include "ris_device.h"
#include "ris_internal.h"

namespace ris {
namespace {

constexpr int kNormThreads = 256;

__device__ __forceinline__ float load_elt(const void* p, int64_t i, bool bf16) {
    return bf16 ? bf16_to_f32(static_cast<const uint16_t*>(p)[i]) : static_cast<const float*>(p)[i];
}
__device__ __forceinline__ void store_elt(void* p, int64_t i, float v, bool bf16) {
    if (bf16)
        static_cast<uint16_t*>(p)[i] = f32_to_bf16(v);
    else
        static_cast<float*>(p)[i] = v;
}

// 16-byte vectors: 8 bf16 or 4 float32 elements.
template <bool BF16> constexpr int kVecElts = BF16 ? 8 : 4;

template <bool BF16>
__device__ __forceinline__ void unpack_vec(u32x4_t v, float* f) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (BF16) {
            f[2 * i] = __uint_as_float(v[i] << 16);
            f[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
        } else {
            f[i] = __uint_as_float(v[i]);
        }
    }
}
template <bool BF16>
__device__ __forceinline__ u32x4_t pack_vec(const float* f) {
    u32x4_t v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (BF16) v[i] = pack_bf16x2(f[2 * i], f[2 * i + 1]);
        else v[i] = __float_as_uint(f[i]);
    }
    return v;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Rows that are no whole, aligned vectors or too long for registers: one
// workgroup per row, element by element.  r = x (+ residual); residual <- r when given (the
// stored value, rounded to the element type, is what the norm reads back, so
// the residual stream and the norm see the same numbers); out = r * rsqrt(mean
// (r^2) + eps) * w.
__global__ __launch_bounds__(kNormThreads) void k_rmsnorm(const void* x, void* residual, const void* w,
                                                          void* out, int64_t cols, float eps, int bf16) {
    __shared__ float red[kNormThreads / 64];
    const int64_t row = blockIdx.x;
    const int64_t base = row * cols;
    float ss = 0.f;
    for (int64_t c = threadIdx.x; c < cols; c += kNormThreads) {
        float r = load_elt(x, base + c, bf16);
        if (residual) {
            r += load_elt(residual, base + c, bf16);
            store_elt(residual, base + c, r, bf16);
            r = load_elt(residual, base + c, bf16);
        }
        ss += r * r;
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < kNormThreads / 64; ++i) tot += red[i];
    const float inv = rsqrtf(tot / (float)cols + eps);
    for (int64_t c = threadIdx.x; c < cols; c += kNormThreads) {
        const float r = residual ? load_elt(residual, base + c, bf16) : load_elt(x, base + c, bf16);
        store_elt(out, base + c, r * inv * load_elt(w, c, bf16), bf16);
    }
}

// The same on rows of whole, aligned 16-byte vectors, to the same bits: thread t
// of the form above adds the squares of the columns t, t + 256, .. in turn, and
// the two forms below keep these chains and the order in which they meet.  A row
// stays in registers as stored (kRegs vectors a lane), so x and residual are
// read once and nothing is read back, and the weights come in beside the row:
// HBM-bound.  32,768 rows of 1,536 bf16 with the residual: 254 us with one
// element per access, 70 us as vectors (5.7 TB/s).

// r[i] <- vector first + i * kStep of x (+ residual, stored back), g[i] <- of w.
template <bool BF16, int kRegs, int kStep>
__device__ __forceinline__ void load_row(const void* x, void* residual, const void* w, int64_t base, int first, int nv,
                                         u32x4_t (&r)[kRegs], u32x4_t (&g)[kRegs]) {
    constexpr int kVec = kVecElts<BF16>;
    u32x4_t* res = static_cast<u32x4_t*>(residual);
    u32x4_t old[kRegs];
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        const int v = first + i * kStep;
        if (v < nv) {
            r[i] = static_cast<const u32x4_t*>(x)[base + v];
            if (residual) old[i] = res[base + v];
            g[i] = static_cast<const u32x4_t*>(w)[v];
        }
    }
    if (!residual) return;
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        const int v = first + i * kStep;
        if (v < nv) {
            float f[kVec], o[kVec];
            unpack_vec<BF16>(r[i], f);
            unpack_vec<BF16>(old[i], o);
#pragma unroll
            for (int e = 0; e < kVec; ++e) f[e] += o[e];
            r[i] = pack_vec<BF16>(f);                 // the norm sees the stored values
            res[base + v] = r[i];
        }
    }
}

template <bool BF16, int kRegs, int kStep>
__device__ __forceinline__ void store_row(void* out, int64_t base, int first, int nv, float inv,
                                          const u32x4_t (&r)[kRegs], const u32x4_t (&g)[kRegs]) {
    constexpr int kVec = kVecElts<BF16>;
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        const int v = first + i * kStep;
        if (v < nv) {
            float f[kVec], y[kVec];
            unpack_vec<BF16>(r[i], f);
            unpack_vec<BF16>(g[i], y);
#pragma unroll
            for (int e = 0; e < kVec; ++e) y[e] = f[e] * inv * y[e];
            static_cast<u32x4_t*>(out)[base + v] = pack_vec<BF16>(y);
        }
    }
}

// 256 / kVec lanes own a row: element e of a lane's vectors (the columns kVec *
// lane + e, then 256 further on, ..) is one chain, kept in the lane.  No barrier.
template <bool BF16, int kRegs>
__global__ __launch_bounds__(kNormThreads, 4)
void k_rmsnorm_lanes(const void* x, void* residual, const void* w, void* out, int64_t rows, int cols, float eps) {
    constexpr int kVec = kVecElts<BF16>;
    constexpr int kLanes = kNormThreads / kVec;       // a row's lanes: 32 bf16, 64 float32
    const int t = threadIdx.x % kLanes;
    const int64_t row = (int64_t)blockIdx.x * (kNormThreads / kLanes) + threadIdx.x / kLanes;
    if (row >= rows) return;                          // all of a row's lanes
    const int nv = cols / kVec;
    const int64_t base = row * nv;
    u32x4_t r[kRegs], g[kRegs];
    load_row<BF16, kRegs, kLanes>(x, residual, w, base, t, nv, r, g);
    float ss[kVec];
#pragma unroll
    for (int e = 0; e < kVec; ++e) ss[e] = 0.f;
#pragma unroll
    for (int i = 0; i < kRegs; ++i)
        if (t + i * kLanes < nv) {
            float f[kVec];
            unpack_vec<BF16>(r[i], f);
#pragma unroll
            for (int e = 0; e < kVec; ++e) ss[e] = fmaf(f[e], f[e], ss[e]);
        }
    // the butterfly of 64 neighbouring chains (wave_sum there), then the four in turn
    float s = (ss[0] + ss[1]) + (ss[2] + ss[3]);
    if constexpr (BF16) s += (ss[4] + ss[5]) + (ss[6] + ss[7]);
    s += dpp<0xB1>(s, 0.0f);                          // quad_perm [1,0,3,2]
    s += dpp<0x4E>(s, 0.0f);                          // quad_perm [2,3,0,1]
    s += dpp<0x141>(s, 0.0f);                         // row_half_mirror
    if constexpr (!BF16) s += dpp<0x140>(s, 0.0f);    // row_mirror
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < kNormThreads / 64; ++i) tot += __shfl(s, i * (64 / kVec), kLanes);
    store_row<BF16, kRegs, kLanes>(out, base, t, nv, rsqrtf(tot / (float)cols + eps), r, g);
}

// A workgroup to a row.  The vectors pass through LDS once, where each thread
// reads its chain's columns.
template <bool BF16, int kRegs>
__global__ __launch_bounds__(kNormThreads, 4)
void k_rmsnorm_wide(const void* x, void* residual, const void* w, void* out, int cols, float eps) {
    constexpr int kVec = kVecElts<BF16>;
    __shared__ u32x4_t vals[kRegs * kNormThreads];
    __shared__ float red[kNormThreads / 64];
    const int t = threadIdx.x, nv = cols / kVec;
    const int64_t base = (int64_t)blockIdx.x * nv;
    u32x4_t r[kRegs], g[kRegs];
    load_row<BF16, kRegs, kNormThreads>(x, residual, w, base, t, nv, r, g);
#pragma unroll
    for (int i = 0; i < kRegs; ++i)
        if (t + i * kNormThreads < nv) vals[t + i * kNormThreads] = r[i];
    __syncthreads();
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < kRegs * kVec; ++k) {
        const int c = t + k * kNormThreads;
        const float f = load_elt(vals, c, BF16);      // past the row: inside vals, and not used
        ss = c < cols ? fmaf(f, f, ss) : ss;
    }
    ss = wave_sum(ss);
    if ((t & 63) == 0) red[t >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < kNormThreads / 64; ++i) tot += red[i];
    store_row<BF16, kRegs, kNormThreads>(out, base, t, nv, rsqrtf(tot / (float)cols + eps), r, g);
}

// Element by element, where rows are no whole, aligned vectors:
// out[r, c] = silu(gu[r, c]) * gu[r, I + c], silu(g) = g / (1 + exp(-g)).
__global__ void k_swiglu(const void* gu, void* out, int64_t rows, int64_t inter, int bf16) {
    const int64_t n = rows * inter;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / inter, c = i - r * inter;
        const float g = load_elt(gu, r * 2 * inter + c, bf16);
        const float u = load_elt(gu, r * 2 * inter + inter + c, bf16);
        store_elt(out, i, g / (1.0f + expf(-g)) * u, bf16);
    }
}


// Whole, aligned 16-byte vectors: two a lane, a workgroup apart so that every
// access of a wave is one contiguous piece, where a tensor goes past the caches:
// HBM-bound, 32,768 rows of 2 x 8,960 bf16 take 286 us (6.2 TB/s) against 770 us
// with 2-byte accesses.  Elsewhere one a lane: small tensors are one latency, which
// two made longer than 2-byte accesses did (32 rows 3.6 us, 3.3 element by element,
// 3.1 here; 2,048 rows 23.4, 47 and 19.6).
constexpr int swiglu_vecs(bool stream) { return stream ? 2 : 1; }
template <bool BF16, bool STREAM>
__global__ __launch_bounds__(256) void k_swiglu_vec(const u32x4_t* gu, u32x4_t* out, uint32_t n, uint32_t vpr) {
    constexpr int kVec = kVecElts<BF16>, kVecs = swiglu_vecs(STREAM);
    const uint32_t i0 = blockIdx.x * (256u * kVecs) + threadIdx.x;
    u32x4_t gv[kVecs], uv[kVecs];
#pragma unroll
    for (int k = 0; k < kVecs; ++k) {
        const uint32_t i = i0 + 256u * k;
        if (i < n) {
            const int64_t at = (int64_t)(i / vpr) * vpr + i;      // row 2 vpr + column
            gv[k] = STREAM ? __builtin_nontemporal_load(gu + at) : gu[at];
            uv[k] = STREAM ? __builtin_nontemporal_load(gu + at + vpr) : gu[at + vpr];
        }
    }
#pragma unroll
    for (int k = 0; k < kVecs; ++k) {
        const uint32_t i = i0 + 256u * k;
        if (i < n) {
            float g[kVec], u[kVec];
            unpack_vec<BF16>(gv[k], g);
            unpack_vec<BF16>(uv[k], u);
#pragma unroll
            for (int e = 0; e < kVec; ++e) g[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
            if (STREAM) __builtin_nontemporal_store(pack_vec<BF16>(g), out + i);
            else out[i] = pack_vec<BF16>(g);
        }
    }
}

// Rows of whole vectors, up to 8,192 bf16 or 4,096 float32 columns.  A workgroup to
// a row has more loads in flight where rows are few (256 rows of 1,536 bf16 with
// the residual: 2.7 against 4.6 us), 32 lanes to a row cost less where they are
// many (16,384 rows of 1,000: 20.8 against 22.6); 64 lanes gain nothing on float32
// rows of more than two vectors a lane (16,384 of 1,536: 60.6 against 63.3).
template <bool BF16>
bool rmsnorm_vec(const void* x, void* residual, const void* w, void* out, int64_t rows, int64_t cols, float eps,
                 hipStream_t st) {
    constexpr int kVec = kVecElts<BF16>, kLanes = kNormThreads / kVec, kPer = kNormThreads / kLanes;
    constexpr int64_t kManyRows = 4096;
    if (cols % kVec != 0 || !aligned16(x) || !aligned16(residual) || !aligned16(w) || !aligned16(out)) return false;
    const int64_t nv = cols / kVec, regs = (nv + kLanes - 1) / kLanes, wide = (nv + kNormThreads - 1) / kNormThreads;
    const dim3 block(kNormThreads);
    const auto lanes = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)((rows + kPer - 1) / kPer)), block, 0, st, x, residual, w, out, rows,
                           (int)cols, eps);
    };
    const auto group = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)rows), block, 0, st, x, residual, w, out, (int)cols, eps);
    };
    if (regs <= 2) lanes(k_rmsnorm_lanes<BF16, 2>);
    else if (BF16 && rows > kManyRows && regs <= 8) {
        if (regs <= 4) lanes(k_rmsnorm_lanes<true, 4>);
        else if (regs <= 6) lanes(k_rmsnorm_lanes<true, 6>);
        else lanes(k_rmsnorm_lanes<true, 8>);
    }
    else if (wide <= 1) group(k_rmsnorm_wide<BF16, 1>);
    else if (wide <= 2) group(k_rmsnorm_wide<BF16, 2>);
    else if (wide <= 3) group(k_rmsnorm_wide<BF16, 3>);
    else if (wide <= 4) group(k_rmsnorm_wide<BF16, 4>);
    else return false;
    return true;
}

// Bytes read and written from which they go past the caches.  At 2 x 8,960 bf16,
// the product that reads the output included: 6,000 rows (323 MB in all) 207 us in
// the caches and 209 past them, 9,000 (484 MB) 268 and 268, 12,000 (645 MB; the
// output alone would still fit the 256 MB last-level cache) 410 and 407, 14,000 456
// and 451, 32,768 926 and 928; the kernel alone 54 and 55, 85 and 81, 111 and 106,
// 129 and 124, 301 and 293.  (Loads or stores alone so: no gain.)
constexpr int64_t kStreamBytes = 512ll << 20;

template <bool BF16, bool STREAM>
void run_swiglu_vec(const void* gu, void* out, int64_t n, int64_t vpr, hipStream_t st) {
    constexpr int64_t kPer = 256 * swiglu_vecs(STREAM);
    hipLaunchKernelGGL((k_swiglu_vec<BF16, STREAM>), dim3((unsigned)((n + kPer - 1) / kPer)), dim3(256), 0, st,
                       static_cast<const u32x4_t*>(gu), static_cast<u32x4_t*>(out), (uint32_t)n, (uint32_t)vpr);
}

template <bool BF16>
bool swiglu_vec(const void* gu, void* out, int64_t rows, int64_t inter, hipStream_t st) {
    constexpr int kVec = kVecElts<BF16>;
    if (inter % kVec != 0 || !aligned16(gu) || !aligned16(out)) return false;
    const int64_t vpr = inter / kVec, n = rows * vpr;
    if (n > 0x7FFFFFFFll) return false;               // 32-bit vector indices
    if (48 * n > kStreamBytes) run_swiglu_vec<BF16, true>(gu, out, n, vpr, st);
    else run_swiglu_vec<BF16, false>(gu, out, n, vpr, st);
    return true;
}

}  // namespace

hipError_t launch_rmsnorm(const void* x, void* residual, const void* w, void* out, int64_t rows,
                          int64_t cols, float eps, int bf16, hipStream_t st) {
    if (bf16 ? rmsnorm_vec<true>(x, residual, w, out, rows, cols, eps, st)
             : rmsnorm_vec<false>(x, residual, w, out, rows, cols, eps, st))
        return hipGetLastError();
    hipLaunchKernelGGL(k_rmsnorm, dim3((unsigned)rows), dim3(kNormThreads), 0, st, x, residual, w, out, cols,
                       eps, bf16);
    return hipGetLastError();
}

hipError_t launch_swiglu(const void* gu, void* out, int64_t rows, int64_t inter, int bf16, hipStream_t st) {
    if (bf16 ? swiglu_vec<true>(gu, out, rows, inter, st) : swiglu_vec<false>(gu, out, rows, inter, st))
        return hipGetLastError();
    const int64_t n = rows * inter;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_swiglu, dim3((unsigned)blocks), dim3(256), 0, st, gu, out, rows, inter, bf16);
    return hipGetLastError();
}

}  // namespace ris
