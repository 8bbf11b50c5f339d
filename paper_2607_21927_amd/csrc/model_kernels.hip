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

// The same on rows of whole, aligned 16-byte vectors (kVec elements).  kWaves
// waves own a row and hold it in registers (kRegs vectors a lane), so x and
// residual are read once and nothing is read back: HBM-bound.  A wave to a row
// needs no barrier; 256 / kWaves / 64 rows share a workgroup.  32,768 rows of
// 1,536 bf16 with the residual: 254 us with one element per access, 70 us as
// vectors (5.7 TB/s).
template <bool BF16, int kWaves, int kRegs>
__global__ __launch_bounds__(kNormThreads) void k_rmsnorm_vec(const void* x, void* residual, const void* w, void* out,
                                                              int64_t rows, int cols, float eps) {
    constexpr int kVec = kVecElts<BF16>;
    constexpr int kRowThreads = 64 * kWaves;
    __shared__ float red[kNormThreads / 64];
    const int t = threadIdx.x % kRowThreads;
    const int64_t row = (int64_t)blockIdx.x * (kNormThreads / kRowThreads) + threadIdx.x / kRowThreads;
    if (row >= rows) return;                          // whole waves, and whole workgroups where waves share a row
    const int nv = cols / kVec;
    const int64_t base = row * nv;
    float r[kRegs][kVec];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        const int v = t + i * kRowThreads;
        if (v < nv) unpack_vec<BF16>(static_cast<const u32x4_t*>(x)[base + v], r[i]);
    }
    if (residual) {
        u32x4_t* res = static_cast<u32x4_t*>(residual);
        u32x4_t old[kRegs];
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            const int v = t + i * kRowThreads;
            if (v < nv) old[i] = res[base + v];
        }
#pragma unroll
        for (int i = 0; i < kRegs; ++i) {
            const int v = t + i * kRowThreads;
            if (v < nv) {
                float o[kVec];
                unpack_vec<BF16>(old[i], o);
#pragma unroll
                for (int e = 0; e < kVec; ++e) r[i][e] += o[e];
                const u32x4_t sum = pack_vec<BF16>(r[i]);
                res[base + v] = sum;
                unpack_vec<BF16>(sum, r[i]);          // the norm sees the stored values
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kRegs; ++i)
        if (t + i * kRowThreads < nv) {
#pragma unroll
            for (int e = 0; e < kVec; ++e) ss += r[i][e] * r[i][e];
        }
    float tot = wave_sum(ss);
    if constexpr (kWaves > 1) {
        static_assert(kWaves == 1 || kWaves * 64 == kNormThreads, "one row per workgroup where waves share it");
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tot;
        __syncthreads();
        tot = 0.f;
#pragma unroll
        for (int i = 0; i < kNormThreads / 64; ++i) tot += red[i];
    }
    const float inv = rsqrtf(tot / (float)cols + eps);
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        const int v = t + i * kRowThreads;
        if (v < nv) {
            float g[kVec];
            unpack_vec<BF16>(static_cast<const u32x4_t*>(w)[v], g);
#pragma unroll
            for (int e = 0; e < kVec; ++e) g[e] = r[i][e] * inv * g[e];
            static_cast<u32x4_t*>(out)[base + v] = pack_vec<BF16>(g);
        }
    }
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


// Whole, aligned 16-byte vectors: a lane takes kSwigluVecs of them, a workgroup
// apart so that every access of a wave is one contiguous piece.  HBM-bound:
// 32,768 rows of 2 x 8,960 bf16 take 352 us (5.0 TB/s, the rate of a device
// copy) against 781 us with 2-byte accesses, and 320 us past the caches.
constexpr int kSwigluVecs = 2;
template <bool BF16, bool STREAM>
__global__ __launch_bounds__(256) void k_swiglu_vec(const u32x4_t* gu, u32x4_t* out, uint32_t n, uint32_t vpr) {
    constexpr int kVec = kVecElts<BF16>;
    const uint32_t i0 = blockIdx.x * (256u * kSwigluVecs) + threadIdx.x;
    u32x4_t gv[kSwigluVecs], uv[kSwigluVecs];
#pragma unroll
    for (int k = 0; k < kSwigluVecs; ++k) {
        const uint32_t i = i0 + 256u * k;
        if (i < n) {
            const int64_t at = (int64_t)(i / vpr) * vpr + i;      // row 2 vpr + column
            gv[k] = STREAM ? __builtin_nontemporal_load(gu + at) : gu[at];
            uv[k] = STREAM ? __builtin_nontemporal_load(gu + at + vpr) : gu[at + vpr];
        }
    }
#pragma unroll
    for (int k = 0; k < kSwigluVecs; ++k) {
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

template <bool BF16, int kWaves>
void run_rmsnorm_vec(int regs, const void* x, void* residual, const void* w, void* out, int64_t rows, int cols,
                     float eps, hipStream_t st) {
    const int64_t per = kNormThreads / (64 * kWaves);
    const dim3 grid((unsigned)((rows + per - 1) / per)), block(kNormThreads);
    switch (regs) {
        case 1: hipLaunchKernelGGL((k_rmsnorm_vec<BF16, kWaves, 1>), grid, block, 0, st, x, residual, w, out, rows, cols, eps); break;
        case 2: hipLaunchKernelGGL((k_rmsnorm_vec<BF16, kWaves, 2>), grid, block, 0, st, x, residual, w, out, rows, cols, eps); break;
        case 3: hipLaunchKernelGGL((k_rmsnorm_vec<BF16, kWaves, 3>), grid, block, 0, st, x, residual, w, out, rows, cols, eps); break;
        default: hipLaunchKernelGGL((k_rmsnorm_vec<BF16, kWaves, 4>), grid, block, 0, st, x, residual, w, out, rows, cols, eps); break;
    }
}

// Rows of whole vectors that four waves' registers can hold (kMaxRegs vectors
// a lane: 8,192 bf16 or 4,096 float32 columns).
constexpr int kMaxRegs = 4;
template <bool BF16>
bool rmsnorm_vec(const void* x, void* residual, const void* w, void* out, int64_t rows, int64_t cols, float eps,
                 hipStream_t st) {
    constexpr int kVec = kVecElts<BF16>;
    if (cols % kVec != 0 || !aligned16(x) || !aligned16(residual) || !aligned16(w) || !aligned16(out)) return false;
    const int64_t nv = cols / kVec;
    if (nv <= 64 * kMaxRegs)
        run_rmsnorm_vec<BF16, 1>((int)((nv + 63) / 64), x, residual, w, out, rows, (int)cols, eps, st);
    else if (nv <= kNormThreads * kMaxRegs)
        run_rmsnorm_vec<BF16, 4>((int)((nv + kNormThreads - 1) / kNormThreads), x, residual, w, out, rows, (int)cols,
                                 eps, st);
    else
        return false;
    return true;
}

// Bytes read and written from which they go past the caches: twice the
// last-level cache (256 MB), so that what the next layer reads is not in it
// anyway.  32,768 rows of 2 x 8,960 bf16 (1.8 GB): 352 against 320 us (loads or
// stores alone so: no gain).
constexpr int64_t kStreamBytes = 512ll << 20;

template <bool BF16>
bool swiglu_vec(const void* gu, void* out, int64_t rows, int64_t inter, hipStream_t st) {
    constexpr int kVec = kVecElts<BF16>;
    if (inter % kVec != 0 || !aligned16(gu) || !aligned16(out)) return false;
    const int64_t vpr = inter / kVec, n = rows * vpr;
    if (n > 0x7FFFFFFFll) return false;               // 32-bit vector indices
    const int64_t per = 256 * kSwigluVecs;
    const dim3 grid((unsigned)((n + per - 1) / per));
    const u32x4_t* g = static_cast<const u32x4_t*>(gu);
    if (48 * n > kStreamBytes)
        hipLaunchKernelGGL((k_swiglu_vec<BF16, true>), grid, dim3(256), 0, st, g, static_cast<u32x4_t*>(out),
                           (uint32_t)n, (uint32_t)vpr);
    else
        hipLaunchKernelGGL((k_swiglu_vec<BF16, false>), grid, dim3(256), 0, st, g, static_cast<u32x4_t*>(out),
                           (uint32_t)n, (uint32_t)vpr);
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
