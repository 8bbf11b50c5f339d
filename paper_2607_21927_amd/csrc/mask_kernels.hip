// Geometry kernels: per-row key sets of the seed ensemble, emitted as CSR.
//
// Each row (kv_head, q) is built by one group of threads: a workgroup, or a
// wave where rows are light.  The row's pool is a
// bitmap in LDS; every (seed, draw) pair of the ensemble is spread over the
// group's lanes, each lane evaluates the keyed permutation and ORs its key into
// the bitmap.
// The bitmap *is* the union over seeds (the paper merges every seed into one
// master set and discards the seed; Methods, "Memory-Bounded Geometry
// Generation"), and reading it in word order yields the row ascending and
// without duplicates (the unique() merge; Methods, "Hybrid Anchor and
// Pre-Fusion Unified Softmax").
//
// Two-pass build: the count pass writes each row's size (popcount) to
// row_ptr[r + 1], a single-workgroup scan turns sizes into offsets, and the
// fill pass regenerates the bitmap and places every key by a group-wide prefix
// over word popcounts; rows are launched in descending q (their cost grows
// with q) so the heavy rows start first.  One-pass build (col_idx sized from
// the closed-form bound): every bitmap is built once and each row's offset found
// by a decoupled look-back, in a persistent grid for heavy rows (k_mask_fused)
// and in chunks of rows for light and for few ones (k_mask_chunk).
#include "ris_device.h"
#include "ris_internal.h"
#include "lookback.h"

namespace ris {
namespace {

constexpr int kThreads = 256;

// A row is built by a group of T threads: one wave (T = 64, several rows to a
// workgroup), or a whole workgroup (T = 256 or 1,024).
template <int T>
__device__ __forceinline__ int group_tid() {
    return T == 64 ? (int)(threadIdx.x & 63u) : (int)threadIdx.x;
}
// Orders the group's LDS accesses.  A wave's LDS operations execute in order,
// so a wave only needs the compiler to keep them so.
template <int T>
__device__ __forceinline__ void group_sync() {
    if constexpr (T == 64) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// Seeds are taken in batches whose row words live in LDS at once: as few
// batches as kSeedBatch allows, of equal size where a wave's are small.  A lane's slice of a batch,
// ceil(seeds * draws / T) draws, is then at most one seed's draws long: it
// spans at most one seed boundary.
template <int T> constexpr int kSeedBatch = T < 256 ? 64 : 256;
static_assert(kSeedBatch<64> <= 64 && kSeedBatch<256> <= 256, "a lane's slice of a batch must not exceed one seed's draws");
template <int T>
__host__ __device__ __forceinline__ int seed_batch(int n_seeds) {
    if constexpr (T == 64) {
        const int n = (n_seeds + kSeedBatch<T> - 1) / kSeedBatch<T>;
        return (n_seeds + n - 1) / n;
    }
    return n_seeds < kSeedBatch<T> ? n_seeds : kSeedBatch<T>;
}

// LDS words of the seed batch's row words.
template <int T>
__host__ __device__ __forceinline__ int64_t rks_words(const MaskParams& p) {
    return (int64_t)seed_batch<T>(p.n_seeds) * kRowWords;
}

// Bitmap words of the largest pool of the built rows: q0 + nq keys (causal)
// or N.
__host__ __device__ __forceinline__ int64_t bitmap_words(const MaskParams& p) {
    const int64_t span = p.causal ? p.q0 + p.nq : p.N;
    return (span + 31) / 32;
}

// LDS words of one group's slice: row words and bitmap, whole 16-byte pieces.
template <int T>
__host__ __device__ __forceinline__ int64_t group_words(const MaskParams& p) {
    return (rks_words<T>(p) + bitmap_words(p) + 3) & ~(int64_t)3;
}

struct RowGeom {
    uint32_t pool;          // draw pool [0, pool)
    uint32_t draws;         // keys per seed
    uint32_t clique_start;  // Structural clique [clique_start, q]
    uint32_t clique_len;
};

__host__ __device__ __forceinline__ RowGeom row_geometry(const MaskParams& p, int64_t q) {
    RowGeom g;
    if (p.mode == 0) {
        const int64_t n = p.causal ? q + 1 : p.N;
        g.pool = (uint32_t)n;
        g.draws = (uint32_t)row_count(p.ppm, n);
        g.clique_start = 0;
        g.clique_len = 0;
    } else {
        const int64_t start = (q / p.block) * (int64_t)p.block;
        const int64_t clique = q - start + 1;
        const int64_t k = row_count(p.ppm, q + 1);
        int64_t kg = k - clique;
        if (kg < 0) kg = 0;
        if (kg > start) kg = start;
        g.pool = (uint32_t)start;
        g.draws = (uint32_t)kg;
        g.clique_start = (uint32_t)start;
        g.clique_len = (uint32_t)clique;
    }
    return g;
}

// Seed index s and draw index j of flat index idx = s * draws + j (idx < 2^24,
// so the float quotient is off by at most one and is corrected).
__device__ __forceinline__ void split_draw(uint32_t idx, uint32_t draws, float inv_draws, int& s, int& j) {
    s = (int)((float)idx * inv_draws);
    j = (int)idx - s * (int)draws;
    if (j < 0) { --s; j += (int)draws; }
    if (j >= (int)draws) { ++s; j -= (int)draws; }
}


// One lane's share of the batch's (seed, draw) pairs, OR-ed into the bitmap.
// Lane t takes the contiguous flat indices [t per, (t+1) per) (flat index =
// seed * draws + draw) and works through them with two walkers held in the
// low and high 16-bit halves of the same registers, so that one packed round
// advances both: walker A takes the lane's draws from the front, walker B
// from the back, until they meet; the lane ends when its last draw is done
// rather than when the slower of two fixed halves is.  A walker's seed -- and
// the round keys it holds -- changes at most a few times per batch.  Each
// walker moves one permutation step per iteration: a walker whose value lands
// in the pool emits it and starts its next draw at once, so cycle walks of
// different lengths do not hold the wave at the slowest lane.  Every walk
// returns to the pool within the domain size (the cycle through j < n returns
// to j), and every iteration advances an unfinished draw, so (slice length)
// * size iterations bound the loop; the bound, from the longest slice, is
// the same in every lane, so the counter lives in scalar registers.
template <int ROUNDS, int T>
__device__ __forceinline__ void walk_draws(const FeistelDomain& dom, const uint32_t* rks,
                                           uint32_t* bits, uint32_t total, uint32_t draws,
                                           float inv_draws) {
    const uint32_t per = (total + T - 1) / T;
    const uint32_t lo = group_tid<T>() * per;
    const uint32_t hi = min(lo + per, total);
    if (lo >= hi) return;
    // Walker A takes the lane's draws from the front, walker B from the back;
    // iA and iB are the flat indices they hold (iB = hi when B never starts),
    // and a walker is done when its next index is the other's.
    bool actA = true, actB = hi - lo >= 2;
    uint32_t iA = lo, iB = actB ? hi - 1u : hi;
    int sA = 0, jA = 0, sB = 0, jB = 0;
    split_draw(lo, draws, inv_draws, sA, jA);
    if (actB) split_draw(hi - 1, draws, inv_draws, sB, jB);
    uint32_t KM[ROUNDS], KX[ROUNDS];
    auto key = [&](int s, int r) -> uint32_t {
        return r < kRowWords ? rks[s * kRowWords + r] : (rks[s * kRowWords + r - kRowWords] ^ kKeyTweak);
    };
    auto load_A = [&]() {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t k = key(sA, r);
            KM[r] = (KM[r] & 0xFFFF0000u) | (k >> 16) | 1u;
            KX[r] = (KX[r] & 0xFFFF0000u) | (k & 0xFFFFu);
        }
    };
    auto load_B = [&]() {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t k = key(sB, r);
            KM[r] = (KM[r] & 0xFFFFu) | (k & 0xFFFF0000u) | 0x10000u;
            KX[r] = (KX[r] & 0xFFFFu) | (k << 16);
        }
    };
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) { KM[r] = 0x00010001u; KX[r] = 0u; }
    load_A();
    if (actB) load_B();
    const uint32_t b = dom.b, mb = (1u << b) - 1u, n = dom.n;
    const u16x2_t sh_a = {(unsigned short)(16u - dom.a), (unsigned short)(16u - dom.a)};
    const u16x2_t sh_b = {(unsigned short)(16u - b), (unsigned short)(16u - b)};
    uint32_t xA = (uint32_t)jA, xB = (uint32_t)jB;
    // per >= hi - lo, and per and the domain size are the same in every lane.
    const uint64_t max_it = (uint64_t)per * dom.size;
    for (uint64_t it = 0; it < max_it; ++it) {
        uint32_t L = (xA >> b) | ((xB >> b) << 16);
        uint32_t R = (xA & mb) | ((xB & mb) << 16);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) feistel_round_x2(L, R, KM[r], KX[r], (r & 1) ? sh_b : sh_a);
        xA = ((L & 0xFFFFu) << b) | (R & 0xFFFFu);
        xB = ((L >> 16) << b) | (R >> 16);
        if (actA && xA < n) {
            atomicOr(&bits[xA >> 5], 1u << (xA & 31u));
            if (iA + 1u == iB) {
                actA = false;
            } else {
                ++iA;
                if (++jA == (int)draws) {
                    jA = 0;
                    ++sA;
                    load_A();
                }
                xA = (uint32_t)jA;
            }
        }
        if (actB && xB < n) {
            atomicOr(&bits[xB >> 5], 1u << (xB & 31u));
            if (iB - 1u == iA) {
                actB = false;
            } else {
                --iB;
                if (jB == 0) {
                    jB = (int)draws;
                    --sB;
                    load_B();
                }
                --jB;
                xB = (uint32_t)jB;
            }
        }
        if (!actA && !actB) break;
    }
}

// The same walk for domains of at most 16 bits (pools of at most 65536 keys,
// fewer than 65536 draws per seed): both walkers' values share one register
// X, A in the low and B in the high 16 bits, so the split into halves and the
// recombination after the rounds are one or two packed instructions each.  J
// holds the two walkers' draw indices within their seeds the same way.  rem
// counts the lane's draws that neither walker has started: a walker that
// finishes a draw takes the next one from its end if rem was positive, and
// stops otherwise (rem may go below zero once both have stopped).  A lane's
// slice spans at most one seed boundary (kSeedBatch <= T): a walker
// that crosses it moves into the other walker's seed and copies that walker's
// round keys from the other half of KM and KX.  The set of draws and each
// draw's walk are those of walk_draws, so the bitmap is identical.
// One step of the lane's count of draws not yet started (never negative):
// true when none was left, else the count drops by one.  A single clamped
// subtract does both: its borrow is the branch's lane mask, and the clamp
// keeps an exhausted count at 0, so the other walker stops at its next draw
// too.
__device__ __forceinline__ bool take_last(int& rem) {
    uint64_t borrow;
    asm volatile("v_sub_co_u32 %0, %1, %2, 1 clamp" : "=v"(rem), "=s"(borrow) : "v"(rem));
    return __builtin_amdgcn_inverse_ballot_w64(borrow);
}

// Walker B's step to the previous draw: the high half of J (B's draw
// index) drops by one; true when it was 0, which the subtract's borrow
// reports as the branch's lane mask (the half then reads 0xFFFF).
__device__ __forceinline__ bool step_down_wraps(uint32_t& J) {
    uint64_t borrow;
    asm volatile("v_sub_co_u32 %0, %1, %2, %3" : "=v"(J), "=s"(borrow) : "v"(J), "s"(0x10000u));
    return __builtin_amdgcn_inverse_ballot_w64(borrow);
}

template <int ROUNDS, int T>
__device__ __forceinline__ void walk_draws16(const FeistelDomain& dom, const uint32_t* rks,
                                             uint32_t* bits, uint32_t total, uint32_t draws,
                                             float inv_draws) {
    const uint32_t per = (total + T - 1) / T;
    const uint32_t lo = group_tid<T>() * per;
    const uint32_t hi = min(lo + per, total);
    if (lo >= hi) return;
    bool actA = true, actB = hi - lo >= 2;
    int rem = (int)(hi - lo) - (actB ? 2 : 1);
    int sA = 0, jA = 0, sB = 0, jB = 0;
    split_draw(lo, draws, inv_draws, sA, jA);
    if (actB) split_draw(hi - 1, draws, inv_draws, sB, jB);
    else { sB = sA; jB = jA; }
    uint32_t KM[ROUNDS], KX[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t ka = r < kRowWords ? rks[sA * kRowWords + r] : (rks[sA * kRowWords + r - kRowWords] ^ kKeyTweak);
        const uint32_t kb = r < kRowWords ? rks[sB * kRowWords + r] : (rks[sB * kRowWords + r - kRowWords] ^ kKeyTweak);
        KM[r] = (kb & 0xFFFF0000u) | (ka >> 16) | 0x00010001u;
        KX[r] = (kb << 16) | (ka & 0xFFFFu);
    }
    const uint32_t b = dom.b, mb = (1u << b) - 1u, n = dom.n;
    const uint32_t mb2 = mb | (mb << 16);
    const u16x2_t shx = {(unsigned short)b, (unsigned short)b};
    const u16x2_t sh_a = {(unsigned short)(16u - dom.a), (unsigned short)(16u - dom.a)};
    const u16x2_t sh_b = {(unsigned short)(16u - b), (unsigned short)(16u - b)};
    uint32_t J = (uint32_t)jA | ((uint32_t)jB << 16);
    uint32_t X = J;
    const uint64_t max_it = (uint64_t)per * dom.size;
    for (uint64_t it = 0; it < max_it; ++it) {
        uint32_t L = as_u32(as_u16x2(X) >> shx);
        uint32_t R = X & mb2;
        asm("" : "+v"(L), "+v"(R));
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) feistel_round_x2(L, R, KM[r], KX[r], (r & 1) ? sh_b : sh_a);
        X = as_u32(as_u16x2(L) << shx) | R;
        if (actA && (X & 0xFFFFu) < n) {
            uint32_t w = __builtin_amdgcn_ubfe(X, 5, 11);
            asm("" : "+v"(w));
            atomicOr(&bits[w], 1u << (X & 31u));
            if (take_last(rem)) {
                actA = false;
            } else {
                ++J;
                if ((J & 0xFFFFu) == draws) {
                    J &= 0xFFFF0000u;
#pragma unroll
                    for (int r = 0; r < ROUNDS; ++r) {
                        KM[r] = __builtin_amdgcn_perm(KM[r], KM[r], 0x03020302u);
                        KX[r] = __builtin_amdgcn_perm(KX[r], KX[r], 0x03020302u);
                    }
                }
                X = __builtin_amdgcn_perm(X, J, 0x07060100u);
            }
        }
        if (actB && (X >> 16) < n) {
            uint32_t w = X >> 21;
            asm("" : "+v"(w));
            atomicOr(&bits[w], 1u << ((X >> 16) & 31u));
            if (take_last(rem)) {
                actB = false;
            } else {
                if (step_down_wraps(J)) {
                    // B's draw index was 0 and its half now reads 0xFFFF:
                    // it continues at draws - 1 of the previous seed
                    J -= (0x10000u - draws) << 16;
#pragma unroll
                    for (int r = 0; r < ROUNDS; ++r) {
                        KM[r] = __builtin_amdgcn_perm(KM[r], KM[r], 0x01000100u);
                        KX[r] = __builtin_amdgcn_perm(KX[r], KX[r], 0x01000100u);
                    }
                }
                X = __builtin_amdgcn_perm(J, X, 0x07060100u);
            }
        }
        if (!actA && !actB) break;
    }
}

// Bits [lo, hi) that fall in word w.
__device__ __forceinline__ uint32_t range_bits(uint32_t w, uint32_t lo, uint32_t hi) {
    const uint32_t b0 = w * 32u, b1 = b0 + 32u;
    const uint32_t a = lo > b0 ? lo : b0, e = hi < b1 ? hi : b1;
    if (a >= e) return 0u;
    const uint32_t n = e - a;
    return (n == 32u ? ~0u : ((1u << n) - 1u)) << (a - b0);
}

// Row words of seed s of row (h, q) into LDS.
__device__ __forceinline__ void store_row_words(const MaskParams& p, int s, int64_t q, int h, uint32_t* dst) {
    uint32_t w[kRowWords];
    row_round_keys(p.seed + (uint64_t)s, (uint64_t)q, (uint64_t)h, (uint64_t)p.layer, w);
    *reinterpret_cast<u32x4_t*>(dst) = u32x4_t{w[0], w[1], w[2], w[3]};
    *reinterpret_cast<u32x4_t*>(dst + 4) = u32x4_t{w[4], w[5], w[6], w[7]};
}

// Fill `bits` (W words, already visible to the whole group) with the union of
// every seed's draws for row (h, q), on top of the local window and the
// initial-token anchor clipped to the pool (above the pool they lie inside the
// Structural clique, which is emitted as a range of its own).  Ends with the
// group's accesses ordered (group_sync).  With `have_words` (one batch of seeds)
// the row words are in rks already.
template <int T>
__device__ void build_row_bitmap(const MaskParams& p, int64_t q, int h, const RowGeom& g,
                                 uint32_t* rks, uint32_t* bits, bool have_words = false) {
    const int tid = group_tid<T>();
    const uint32_t W = (g.pool + 31u) >> 5;
    // (The persistent grid has no scalar registers to spare for the choice.)
    if (T == 256 || (p.window | p.anchor) != 0) {
        const uint32_t qe = (uint32_t)q + 1u;
        const uint32_t a_hi = min((uint32_t)p.anchor, min(qe, g.pool));
        const uint32_t w_lo = p.window > 0 && (uint32_t)p.window < qe ? qe - (uint32_t)p.window : 0u;
        const uint32_t w_hi = p.window > 0 ? min(qe, g.pool) : 0u;
        for (uint32_t w = tid; w < W; w += T) bits[w] = range_bits(w, 0u, a_hi) | range_bits(w, w_lo, w_hi);
    } else {
        for (uint32_t w = tid; w < W; w += T) bits[w] = 0u;
    }
    if (g.draws == 0) {
        group_sync<T>();
        return;
    }
    const FeistelDomain dom = make_domain(g.pool);
    const float inv_draws = 1.0f / (float)g.draws;
    // Batches keep the flat (seed, draw) index below 2^24 for the float split.
    const int batch = (int)min((uint32_t)(T == 64 ? seed_batch<T>(p.n_seeds) : kSeedBatch<T>), (1u << 24) / g.draws);
    for (int s0 = 0; s0 < p.n_seeds; s0 += batch) {
        const int sb = min(batch, p.n_seeds - s0);
        group_sync<T>();   // bitmap cleared / previous batch's keys no longer read
        // Row words of the batch's seeds, one Philox evaluation per lane.
        if (!have_words || s0 > 0) {
            for (int t = tid; t < sb; t += T) store_row_words(p, s0 + t, q, h, &rks[t * kRowWords]);
        }
        group_sync<T>();
        const uint32_t total = (uint32_t)sb * g.draws;
        if (dom.size <= 65536u && g.draws < 65536u) {
            if (dom.rounds == 6)
                walk_draws16<6, T>(dom, rks, bits, total, g.draws, inv_draws);
            else
                walk_draws16<12, T>(dom, rks, bits, total, g.draws, inv_draws);
        } else {
            walk_draws<6, T>(dom, rks, bits, total, g.draws, inv_draws);
        }
    }
    group_sync<T>();
}

// Sum of v over the group.
template <int T>
__device__ __forceinline__ uint32_t group_sum(uint32_t v, uint32_t* red) {
    v = wave_sum_u32(v);
    if constexpr (T == 64) return v;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) red[wid] = v;
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) t += red[w];
    __syncthreads();
    return t;
}

// Exclusive prefix of v over the group; *total receives the group's sum.
template <int T>
__device__ __forceinline__ uint32_t group_exclusive_scan(uint32_t v, uint32_t* red, uint32_t* total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan(v);
    if constexpr (T == 64) {
        *total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        return inc - v;
    }
    if (lane == 63) red[wid] = inc;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
        before += w < wid ? red[w] : 0u;
        sum += red[w];
    }
    *total = sum;
    __syncthreads();
    return before + inc - v;
}

// Write the row: the set bits of bits[0, W) as keys 32 w + b, ascending, at
// out[0, ..), then the Structural clique; nothing at out[limit] or beyond.
// A lane's keys of one word are contiguous in out, so it writes them four at
// a time with 16-byte stores (global stores need only 4-byte alignment) and
// the last one to three with an 8- and a 4-byte store: the store
// instructions, whose address processing limits this loop, are about a
// quarter of one key per store.
template <int T>
__device__ void emit_row(const uint32_t* bits, uint32_t W, int32_t* out, int64_t limit, uint32_t clique_start,
                         uint32_t clique_len, uint32_t* red, int64_t count) {
    // The whole row fits below limit in every valid build; the guarded path
    // is for a truncated or inconsistent row_ptr.
    const bool whole = limit >= count;
    uint32_t done = 0;
    for (uint32_t w0 = 0; w0 < W; w0 += T) {
        const uint32_t w = w0 + group_tid<T>();
        uint32_t word = w < W ? bits[w] : 0u;
        uint32_t total;
        const uint32_t pos0 = done + group_exclusive_scan<T>(__popc(word), red, &total);
        const int32_t k0 = (int32_t)(w * 32u);
        auto next_key = [&]() {
            const uint32_t b = (uint32_t)__builtin_ctz(word);   // v_ffbl_b32 (word != 0 here)
            word &= word - 1u;
            return k0 + (int32_t)b;
        };
        // Groups of four keys as 16-byte stores at any 4-byte-aligned position,
        // then the last one to three keys.
        if (whole) {
            int32_t* o = out + pos0;
            for (uint32_t n = __popc(word); n >= 4u; n -= 4u) {
                const int32_t a = next_key(), b = next_key(), c = next_key(), d = next_key();
                *reinterpret_cast<int4*>(o) = make_int4(a, b, c, d);
                o += 4;
            }
            if (__popc(word) >= 2) {
                const int32_t a = next_key(), b = next_key();
                *reinterpret_cast<int2*>(o) = make_int2(a, b);
                o += 2;
            }
            if (word) *o = next_key();
        } else {
            int64_t pos = pos0;
            while (__popc(word) >= 4) {
                const int32_t a = next_key(), b = next_key(), c = next_key(), d = next_key();
                if (pos + 4 <= limit) {
                    *reinterpret_cast<int4*>(out + pos) = make_int4(a, b, c, d);
                } else {
                    if (pos < limit) out[pos] = a;
                    if (pos + 1 < limit) out[pos + 1] = b;
                    if (pos + 2 < limit) out[pos + 2] = c;
                }
                pos += 4;
            }
            if (__popc(word) >= 2) {
                const int32_t a = next_key(), b = next_key();
                if (pos + 2 <= limit) {
                    *reinterpret_cast<int2*>(out + pos) = make_int2(a, b);
                } else if (pos < limit) {
                    out[pos] = a;
                }
                pos += 2;
            }
            if (word) {
                const int32_t k = next_key();
                if (pos < limit) out[pos] = k;
                ++pos;
            }
        }
        done += total;
    }
    for (uint32_t t = group_tid<T>(); t < clique_len; t += T) {
        const int64_t pos = (int64_t)done + t;
        if (pos < limit) out[pos] = (int32_t)(clique_start + t);
    }
}

// Set bits of the row's W words, over the group.
template <int T>
__device__ __forceinline__ uint32_t row_popcount(const uint32_t* bits, uint32_t W, uint32_t* red) {
    uint32_t c = 0;
    for (uint32_t w = group_tid<T>(); w < W; w += T) c += __popc(bits[w]);
    return group_sum<T>(c, red);
}

// The group's index in the launch: a workgroup for T = 256, a wave for T = 64
// (uniform, so that the row's arithmetic is scalar).
template <int T>
__device__ __forceinline__ int64_t group_index() {
    if constexpr (T == 64)
        return (int64_t)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    return blockIdx.x;
}

// The group's LDS slice: the seed batch's row words, then the row's bitmap.
template <int T>
__device__ __forceinline__ uint32_t* group_smem(const MaskParams& p, uint32_t* smem) {
    if constexpr (T == 64)
        return smem + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) * group_words<T>(p);
    return smem;
}

// Group -> (row r, query q, head h), heavy (late) rows first; false past the last row.
__device__ __forceinline__ bool row_of_group(const MaskParams& p, int64_t i, int64_t& r, int64_t& q, int& h) {
    const int64_t local = p.nq - 1 - i / p.heads;
    h = (int)(i % p.heads);
    q = p.q0 + local;
    r = (int64_t)h * p.nq + local;
    return local >= 0;
}

template <int T>
__global__ __launch_bounds__(kThreads) void k_mask_count(MaskParams p, int64_t* row_ptr) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ uint32_t red[kThreads / 64];
    uint32_t* rks = group_smem<T>(p, smem);
    uint32_t* bits = rks + rks_words<T>(p);
    int64_t r, q; int h;
    if (!row_of_group(p, group_index<T>(), r, q, h)) return;      // a whole wave
    const RowGeom g = row_geometry(p, q);
    build_row_bitmap<T>(p, q, h, g, rks, bits);
    const uint32_t total = row_popcount<T>(bits, (g.pool + 31u) >> 5, red);
    if (group_tid<T>() == 0) row_ptr[r + 1] = (int64_t)total + g.clique_len;
}

template <int T>
__global__ __launch_bounds__(kThreads) void k_mask_fill(MaskParams p, const int64_t* row_ptr,
                                                        int32_t* col_idx, int64_t capacity) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ uint32_t red[kThreads / 64];
    uint32_t* rks = group_smem<T>(p, smem);
    uint32_t* bits = rks + rks_words<T>(p);
    int64_t r, q; int h;
    if (!row_of_group(p, group_index<T>(), r, q, h)) return;      // a whole wave
    const int64_t base = row_ptr[r];
    int64_t limit = row_ptr[r + 1] - base;
    // Never write outside col_idx[0, capacity), whatever row_ptr holds.
    if (base < 0 || limit < 0 || base > capacity) return;
    if (limit > capacity - base) limit = capacity - base;
    const RowGeom g = row_geometry(p, q);
    build_row_bitmap<T>(p, q, h, g, rks, bits);
    const uint32_t W = (g.pool + 31u) >> 5;
    const int64_t count = (int64_t)row_popcount<T>(bits, W, red) + g.clique_len;
    emit_row<T>(bits, W, col_idx + base, limit, g.clique_start, g.clique_len, red, count);
}

// ---------------------------------------------------------------------------
// A block-uniform 64-bit value held in scalar registers.
__device__ __forceinline__ int64_t uniform_i64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// One-pass build (count, scan and fill fused), used when col_idx is sized from
// the closed-form bound.  Workgroups take tickets -- a row or a chunk of rows
// each, in row order -- and build each row's
// bitmap once.  A row's offset is
// found by a decoupled look-back over its predecessors' status words, which
// live in row_ptr itself (the protocol and its flags are in lookback.h).  In the
// persistent grid (k_mask_fused) a workgroup publishes a row's size as soon as its bitmap is built and keeps
// the bitmap in LDS while it builds the next rows; it looks back for the row's
// offset (64 predecessors per step, one per lane) and writes its keys only
// after up to two more rows, when the predecessors, whose rows were taken
// earlier, have almost always published their sizes.  Every wait ends: a
// row is held only by a running workgroup, and a workgroup waits only for
// rows below the one it resolves, each of which its holder builds and
// publishes after waits for still smaller rows (induction over the rows).
// The wait is bounded anyway (p.spin_limit
// polls): past the bound the row publishes poison and writes nothing, any row
// whose look-back reaches a poisoned prefix does the same, and k_strip_status
// makes the total row_ptr[R] negative, so that an incomplete CSR is reported
// rather than used.  Status words are read and written with relaxed
// agent-scope atomics: they carry the only data exchanged.
__device__ __forceinline__ int64_t status_load(const int64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(int64_t* p, int64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A row of the persistent build whose size is published but whose keys are not
// yet written: its bitmap waits in LDS until its offset is known, and so does
// this (registers that hold it through the walk cost 1-2% in spills).
struct PendingRow {
    uint32_t row, count;         // rows and their sizes are below 2^31
    uint32_t pool, clique_len;   // the clique, if any, starts at the pool's end
};

// Decoupled look-back, by one whole wave: the number of entries before unit j
// (a row, or a chunk of rows), whose predecessors' statuses lie `stride` entries
// of row_ptr apart (unit i's at row_ptr[(i + 1) * stride]).  Each step covers 64
// predecessors, one per lane, and ends at the nearest one whose inclusive
// prefix is known, once every one before it is ready.  Returns -1 when the
// wait gave up or met poison.
__device__ __forceinline__ int64_t look_back(const MaskParams& p, const int64_t* row_ptr, int64_t j, int stride) {
    namespace lb = lookback;
    const int lane = threadIdx.x & 63;
    int64_t prefix = 0;
    uint32_t spins = 0;
    while (j > 0) {
        const int64_t idx = j - lane;                       // unit idx-1's status
        int64_t v = idx > 0 ? status_load(&row_ptr[idx * stride]) : lb::inclusive(0, false);
        int first;
        for (;;) {
            const uint64_t inc = __ballot(lb::is_inclusive(v));
            first = lb::step_end(inc, __ballot(lb::is_ready(v)));
            if (first >= 0) break;
            if (spins++ >= p.spin_limit) return -1;
            __builtin_amdgcn_s_sleep(1);
            // Only the statuses still missing, up to the nearest inclusive
            // one, are read again: the polls' traffic slows the others.
            if (!lb::is_ready(v) && (inc == 0 || lane < __builtin_ctzll(inc))) v = status_load(&row_ptr[idx * stride]);
        }
        // Lanes before `first` hold single units' counts (their sum stays below
        // 2^32); lane `first` holds an inclusive prefix, or poison.
        prefix += (int64_t)wave_sum_u32(lane < first ? (uint32_t)lb::value(v) : 0u);
        if (first < 64) {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, first);
            const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)v >> 32), first);
            const int64_t vf = (int64_t)(((uint64_t)hi << 32) | lo);
            return lb::is_poisoned(vf) ? -1 : prefix + lb::value(vf);
        }
        j -= 64;
    }
    return prefix;
}

// Find the offset of row x.row, publish its inclusive prefix and write its
// keys.  Block-wide; starts and ends with every thread of the block present.
// x lies in LDS, written by thread 0: the first wave may read it at once, the
// others from the barrier on.
__device__ void resolve_and_emit(const MaskParams& p, int64_t* row_ptr, int32_t* col_idx, int64_t capacity,
                                 const PendingRow& x, const uint32_t* bits, uint32_t* red, int64_t* s_base) {
    namespace lb = lookback;
    if (threadIdx.x < 64) {
        const int64_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)x.row);
        // the test hook's row: as if its wait had given up
        const int64_t prefix = row == p.poison_row ? -1 : look_back(p, row_ptr, row, 1);
        if (threadIdx.x == 0) {
            status_store(&row_ptr[row + 1], lb::inclusive(prefix + (int64_t)x.count, prefix < 0));
            *s_base = prefix;
        }
    }
    __syncthreads();
    const int64_t base = uniform_i64(*s_base);
    if (base >= 0 && base <= capacity) {
        const auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
        const int64_t count = uniform(x.count);
        int64_t limit = count;
        if (limit > capacity - base) limit = capacity - base;
        const uint32_t pool = uniform(x.pool);
        emit_row<kThreads>(bits, (pool + 31u) >> 5, col_idx + base, limit, pool, uniform(x.clique_len), red, count);
    }
}

// One-pass build by chunks: a workgroup takes one ticket -- kRows consecutive
// rows, one per group of T threads --, builds their bitmaps, publishes the
// chunk's size, finds its offset by the look-back over the chunks before it
// and writes the rows.  The chunk's status is the row_ptr entry of its last
// row; the entries of its other rows are written at once as they stay.
// With `fold` the last workgroup to finish strips the statuses (the count of
// finished workgroups lives in the high half of row_ptr[0], the tickets in the
// low one); otherwise the last ticket restores row_ptr[0].
template <int T, int kRows>
__global__ __launch_bounds__(T * kRows, 8) void k_mask_chunk(MaskParams p, int64_t* row_ptr, int32_t* col_idx,
                                                         int64_t capacity, int fold) {
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ uint32_t red[T * kRows / 64], s_count[kRows];
    __shared__ int64_t s_ticket, s_base;
    __shared__ int s_last;
    namespace lb = lookback;
    const int64_t R = (int64_t)p.heads * p.nq;
    const int grp = kRows == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)(threadIdx.x / T));
    uint32_t* rks = smem + (int64_t)grp * group_words<T>(p);
    uint32_t* bits = rks + rks_words<T>(p);
    if (threadIdx.x == 0) {
        const unsigned long long t = atomicAdd(reinterpret_cast<unsigned long long*>(row_ptr), 1ull);
        s_ticket = (int64_t)(uint32_t)t;
        if (!fold && t == (unsigned long long)gridDim.x - 1) status_store(row_ptr, 0);
    }
    __syncthreads();
    const int64_t chunk = uniform_i64(s_ticket);
    const int64_t r0 = chunk * kRows, r = r0 + grp;
    const int rows = (int)(R - r0 < kRows ? R - r0 : kRows);      // rows of this chunk
    // One batch of seeds: the row words of all the chunk's (row, seed) pairs,
    // spread over the workgroup's lanes (a row of 10 seeds alone would leave 54
    // of its wave's 64 lanes idle through the Philox rounds).
    const bool shared_words = T == 64 && p.n_seeds <= kSeedBatch<T>;
    if (shared_words) {
        for (int t = threadIdx.x; t < rows * p.n_seeds; t += T * kRows) {
            const int i = t / p.n_seeds, sd = t - i * p.n_seeds;
            const int h = (int)((r0 + i) / p.nq);
            store_row_words(p, sd, p.q0 + (r0 + i - (int64_t)h * p.nq), h,
                            smem + i * group_words<T>(p) + sd * kRowWords);
        }
        __syncthreads();
    }
    RowGeom g = {};
    uint32_t W = 0;
    int64_t count = 0;
    if (grp < rows) {
        const int h = (int)(r / p.nq);
        const int64_t q = p.q0 + (r - (int64_t)h * p.nq);
        g = row_geometry(p, q);
        W = (g.pool + 31u) >> 5;
        build_row_bitmap<T>(p, q, h, g, rks, bits, shared_words);
        count = (int64_t)__builtin_amdgcn_readfirstlane((int)row_popcount<T>(bits, W, red)) + g.clique_len;
        if (group_tid<T>() == 0) s_count[grp] = (uint32_t)count;
    }
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const uint32_t c = i < rows ? s_count[i] : 0u;
        before += i < grp ? c : 0u;
        total += c;
    }
    if (threadIdx.x < 64) {
        int64_t* status = &row_ptr[r0 + rows];
        if (threadIdx.x == 0) status_store(status, lb::aggregate(total));
        const int64_t prefix = look_back(p, row_ptr, chunk, kRows);
        // the test hook's row poisons itself and what follows
        const bool hook = p.poison_row >= r0 && p.poison_row < r0 + rows;
        if (threadIdx.x == 0) {
            status_store(status, lb::inclusive(prefix + total, prefix < 0 || hook));
            s_base = prefix;
        }
    }
    __syncthreads();
    const int64_t first = uniform_i64(s_base);
    const bool bad = first < 0 || (p.poison_row >= r0 && p.poison_row <= r);
    if (grp < rows) {
        const int64_t base = first + before;
        if (group_tid<T>() == 0 && grp + 1 < rows) status_store(&row_ptr[r + 1], bad ? -1 : base + count);
        if (!bad && base <= capacity) {
            int64_t limit = count;
            if (limit > capacity - base) limit = capacity - base;
            emit_row<T>(bits, W, col_idx + base, limit, g.clique_start, g.clique_len, red, count);
        }
    }
    if (!fold) return;
    if (threadIdx.x == 0) {
        // this thread wrote the chunk's status (through to memory): done before the count
        __builtin_amdgcn_s_waitcnt(0);
        const uint64_t old = __hip_atomic_fetch_add(reinterpret_cast<uint64_t*>(row_ptr), 1ull << 32,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_last = (old >> 32) == (uint64_t)gridDim.x - 1;
    }
    __syncthreads();
    if (!s_last) return;                                      // the same in every thread
    const int any = __syncthreads_or(lb::strip_units(
        threadIdx.x, T * kRows, gridDim.x, kRows, R, [&](int64_t at) { return status_load(&row_ptr[at]); },
        [&](int64_t at, int64_t v) { status_store(&row_ptr[at], v); }));
    if (threadIdx.x == 0) {
        status_store(&row_ptr[R], lb::total_entry(status_load(&row_ptr[R]), any));
        status_store(row_ptr, 0);
    }
}

// Persistent one-pass build.  Every workgroup takes rows (a ticket each,
// in row order) until none is left.  It
// publishes a row's size as soon as the row's
// bitmap is built, but looks back for the row's offset only after building
// kDepth more rows: by then its predecessors have almost always published
// their sizes, so the look-back rarely waits (kDepth = 0: at once).
// kDepth + 1 bitmaps per workgroup rotate through the rows.
template <int kDepth>
__global__ __launch_bounds__(kThreads, kDepth == 2 ? 6 : 8) void k_mask_fused(MaskParams p, int64_t* row_ptr,
                                                                             int32_t* col_idx, int64_t capacity) {
    static_assert(kDepth >= 0 && kDepth <= 2, "at most two rows wait for their offsets");
    extern __shared__ __align__(16) uint32_t smem[];
    __shared__ int64_t s_ticket;
    __shared__ PendingRow ring[kDepth + 1];
    namespace lb = lookback;
    // The row words are dead between a walk and the next row's: the reductions'
    // and the offset's words live there (a few bytes more of LDS cost the 64k
    // layer's sixth workgroup per CU, and 3.5% of the build).
    uint32_t* red = smem;
    int64_t* s_base = reinterpret_cast<int64_t*>(smem + kThreads / 64);
    static_assert(kThreads / 64 + 2 <= kRowWords, "one seed's row words hold both");
    const uint32_t first_at = (uint32_t)rks_words<kThreads>(p), bw = (uint32_t)bitmap_words(p);
    const int64_t R = (int64_t)p.heads * p.nq;
    int waiting = 0, in = 0, out = 0;      // rows that wait; the ring's next entry to fill and to resolve
    bool more = true;
    for (;;) {
        // Every workgroup takes tickets until one is past the rows, so R +
        // gridDim.x are taken in all, and the last one restores row_ptr[0] to 0.
        if (more && threadIdx.x == 0) {
            const int64_t t = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(row_ptr), 1ull);
            s_ticket = t;
            if (t == R + (int64_t)gridDim.x - 1) status_store(row_ptr, 0);
        }
        __syncthreads();   // also: last iteration's bitmap, offset and ring entry are no longer read
        if (more) {
            const int64_t r = uniform_i64(s_ticket);
            more = r < R;
            if (more) {
                const int h = (int)(r / p.nq);
                const int64_t q = p.q0 + (r - (int64_t)h * p.nq);
                const RowGeom g = row_geometry(p, q);
                const uint32_t at = first_at + in * bw;
                build_row_bitmap<kThreads>(p, q, h, g, smem, smem + at);
                const uint32_t W = (g.pool + 31u) >> 5;
                const uint32_t count = row_popcount<kThreads>(smem + at, W, red) + g.clique_len;
                if (threadIdx.x == 0) {
                    status_store(&row_ptr[r + 1], lb::aggregate(count));
                    ring[in] = {(uint32_t)r, count, g.pool, g.clique_len};
                }
                in = in == kDepth ? 0 : in + 1;
                ++waiting;
            }
        }
        if (waiting > (more ? kDepth : 0)) {
            resolve_and_emit(p, row_ptr, col_idx, capacity, ring[out], smem + first_at + out * bw, red, s_base);
            out = out == kDepth ? 0 : out + 1;
            --waiting;
        } else if (!more) {
            break;
        }
    }
}

// Clear row_ptr[0] and the status entries of `units` units of `stride` rows each.
__global__ void k_clear_status(int64_t* row_ptr, int64_t R, int64_t units, int stride) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= units) row_ptr[i * stride < R ? i * stride : R] = 0;
}

// After the one-pass build: strip the flags of the units' status entries.  A
// poisoned entry becomes -1; if any is poisoned, row_ptr[R] becomes
// -1 as well.  row_ptr[0] is 0 when this runs (the last ticket restores it);
// here it counts finished workgroups (low 32 bits) and poisoned
// ones (high bits), and the last workgroup to finish resets it to 0.
__global__ __launch_bounds__(256) void k_strip_status(int64_t* row_ptr, int64_t R, int64_t units, int stride) {
    const int64_t i = 1 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool poison = false;
    if (i <= units) {
        const int64_t at = i * stride < R ? i * stride : R;
        const int64_t v = row_ptr[at];
        poison = lookback::is_poisoned(v);
        // through to memory, and done before the count below: the total's -1 must be the last write
        status_store(&row_ptr[at], lookback::stripped(v));
        __builtin_amdgcn_s_waitcnt(0);
    }
    const int any = __syncthreads_or(poison);
    if (threadIdx.x == 0) {
        const uint64_t add = 1ull | (any ? (1ull << 32) : 0ull);
        const uint64_t old = __hip_atomic_fetch_add(reinterpret_cast<uint64_t*>(row_ptr), add,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((old & 0xFFFFFFFFull) == (uint64_t)gridDim.x - 1) {
            // every other workgroup has stripped its entries
            if (((old + add) >> 32) != 0) status_store(&row_ptr[R], -1);
            status_store(row_ptr, 0);
        }
    }
}

// In-place inclusive scan of row_ptr[1 .. R] (row sizes -> end offsets);
// row_ptr[0] = 0.  One workgroup walks the array in coalesced chunks.
constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;

__global__ __launch_bounds__(kScanThreads) void k_scan_rows(int64_t* row_ptr, int64_t R) {
    __shared__ int64_t wave_tot[kScanThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int64_t carry = 0;
    if (tid == 0) row_ptr[0] = 0;
    for (int64_t base = 1; base <= R; base += (int64_t)kScanThreads * kScanItems) {
        int64_t v[kScanItems];
        int64_t run = 0;
#pragma unroll
        for (int e = 0; e < kScanItems; ++e) {
            const int64_t idx = base + (int64_t)tid * kScanItems + e;
            run += idx <= R ? row_ptr[idx] : 0;
            v[e] = run;
        }
        int64_t inc = run;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t t = __shfl_up(inc, off);
            if (lane >= off) inc += t;
        }
        if (lane == 63) wave_tot[wid] = inc;
        __syncthreads();
        int64_t before = carry;
        int64_t chunk = 0;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            if (w < wid) before += wave_tot[w];
            chunk += wave_tot[w];
        }
        before += inc - run;
#pragma unroll
        for (int e = 0; e < kScanItems; ++e) {
            const int64_t idx = base + (int64_t)tid * kScanItems + e;
            if (idx <= R) row_ptr[idx] = before + v[e];
        }
        carry += chunk;
        __syncthreads();
    }
}

size_t mask_smem_bytes(const MaskParams& p, int bitmaps = 1) {
    return (size_t)(rks_words<kThreads>(p) + bitmaps * bitmap_words(p)) * sizeof(uint32_t);
}
// `groups` groups of T threads, one row each.
template <int T>
size_t group_smem_bytes(const MaskParams& p, int groups) {
    return (size_t)(groups * group_words<T>(p)) * sizeof(uint32_t);
}

// Workgroups per CU below which a deeper one-pass pipeline costs more
// occupancy than its shorter waits gain.
constexpr int kMinResidentRows = 6;
// Rows of fewer expected draws may be built by a wave each (one_pass_form and
// two_phase_waves say where).  A workgroup to such a row spends most of its time
// between barriers and, in the persistent grid, takes a ticket per row (12.5 ns
// each on MI355X, whatever the row's work): 32k layers of 10 seeds
// (1,640 draws) 608 -> 340 us, an 8k layer of 70 (2,870) 211 -> 170, a 4k layer
// of 10 90 -> 34; 4,900 draws 949 -> 702, 6,600 2,188 -> 1,932, 9,800 2,735 ->
// 2,660.  From there the LDS of a bitmap per wave leaves too few waves (11,500
// draws 1,537 -> 1,548, 23,000 4,980 -> 5,550).
constexpr int64_t kWaveDraws = 9000;
// Rows (waves) per workgroup: 8 up to this many draws, where fewer, larger
// chunks shorten the look-back (4k layer 34 against 45 us with 4), 4 above (a
// chunk waits for its slowest row: 6,600 draws 1,932 against 2,021 with 8) and
// where eight bitmaps would leave one workgroup to a CU (100,000 keys: 1,106
// against 1,550 us).
constexpr int64_t kChunk8Draws = 4000;
constexpr size_t kChunk8Smem = 80 << 10;
// Pools of 160,000 keys and more (four bitmaps over 80 KB, one workgroup of four
// waves to a CU) go to the persistent grid: 262,144 keys, 6,600 draws 8.0
// against 13.6 ms.  The two-phase build's waves end at 65,536 keys: further on some
// builds gain 15% and others lose as much or more (101,000 keys, 8,184 rows of 70
// seeds 200 us against 140; 106,000 keys, 4,376 rows of 10 seeds 33 against 27).
constexpr size_t kWaveSmem = 80 << 10;
constexpr int64_t kWaveKeysTwoPhase = 65536;
// A dispatch holds fewer than 2^32 work-items: builds of more rows, 64 or 256 lanes
// each (in chunks of up to 8 rows), go to the persistent grid, whose size does not
// grow with them.
constexpr int64_t kMaxItems = (1ll << 32) - 512;
// Builds of at most this many rows leave CUs idle with 256 lanes to a row; 1,024
// lanes take a row of 46,000 draws in 29 instead of 47 us (2 rows; 512 rows of
// the same 63 instead of 75, 1,024 rows 109 against 105).  Lighter rows gain less
// than the larger workgroup's barriers cost, and so do rows light in each batch of
// seeds: rows of 640 to 2,560 draws take 0.59 of the persistent grid's time with 256
// lanes and 0.65 with 1,024, of 2,600 and more 0.69 and 0.63.
constexpr int64_t kFewRows = 512;
constexpr double kFewRowsDraws = 4000;

template <int kDepth>
hipError_t fused_occupancy(const MaskParams& p, int* blocks) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, k_mask_fused<kDepth>, kThreads,
                                                        mask_smem_bytes(p, kDepth + 1));
}

// Expected draws of the middle row; in Structural mode an upper bound, since the
// clique's length comes off every row's draws (the crossovers above are those of
// Stochastic rows).
int64_t middle_draws(const MaskParams& p) {
    const int64_t mid = p.q0 + p.nq / 2;
    return (int64_t)p.n_seeds * row_count(p.ppm, p.causal ? mid + 1 : p.N);
}

hipError_t clear_status(int64_t* row_ptr, int64_t rows, int64_t units, int stride, hipStream_t st) {
    hipLaunchKernelGGL(k_clear_status, dim3((unsigned)((units + 1 + 255) / 256)), dim3(256), 0, st, row_ptr, rows,
                       units, stride);
    return hipGetLastError();
}
hipError_t strip_status(int64_t* row_ptr, int64_t rows, int64_t units, int stride, hipStream_t st) {
    hipLaunchKernelGGL(k_strip_status, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st, row_ptr, rows, units,
                       stride);
    return hipGetLastError();
}

// Chunks up to which the build's last workgroup strips the statuses itself.
constexpr int64_t kFoldChunks = 1024;

template <int T, int kRows>
hipError_t run_mask_chunk(const MaskParams& p, int64_t* row_ptr, int32_t* col_idx, int64_t capacity, hipStream_t st) {
    const int64_t rows = (int64_t)p.heads * p.nq, chunks = (rows + kRows - 1) / kRows;
    hipError_t e = clear_status(row_ptr, rows, chunks, kRows, st);
    if (e != hipSuccess) return e;
    const int fold = chunks <= kFoldChunks;
    hipLaunchKernelGGL((k_mask_chunk<T, kRows>), dim3((unsigned)chunks), dim3(T * kRows),
                       group_smem_bytes<T>(p, kRows), st, p, row_ptr, col_idx, capacity, fold);
    e = hipGetLastError();
    if (e != hipSuccess || fold) return e;
    return strip_status(row_ptr, rows, chunks, kRows, st);
}

// A seed's draws in the build's rows: of the middle row, of the heaviest, and the
// share of rows that draw at all.
struct RowDraws {
    double mean, most, share;
};
RowDraws row_draws(const MaskParams& p) {
    const int64_t mid = p.q0 + p.nq / 2, last = p.q0 + p.nq - 1;
    const int64_t k_mid = row_count(p.ppm, p.causal ? mid + 1 : p.N);
    if (p.mode == 0) return {(double)k_mid, (double)row_count(p.ppm, p.causal ? last + 1 : p.N), 1.0};
    // A block's rows draw k - 1, k - 2, .. keys, the clique's length less each, down
    // to none: the heaviest is the first row or that of the last block.
    int64_t most = row_geometry(p, p.q0).draws;
    const int64_t start = last / p.block * p.block;
    if (start >= p.q0 && row_geometry(p, start).draws > most) most = row_geometry(p, start).draws;
    if (most == 0) return {0.0, 0.0, 0.0};
    const double n = (double)(k_mid - 1 < p.block ? k_mid - 1 : p.block);
    return {n > 0.0 ? (n * (double)k_mid - n * (n + 1.0) / 2.0) / p.block : 0.0, (double)most,
            most < p.block ? (double)most / p.block : 1.0};
}

// What a form's build takes, in us: the heaviest row's batches of seeds one after the
// other, each with Philox evaluations and a walk (the draws of a lane), and what the
// rows together keep the chip with.  One-pass rows are taken head by head, light to
// heavy, and a head's first ones wait for the offsets of the last head's heaviest.
// Fitted to 6,000 builds of 1 to 300,000 rows, 1 to 1,200 seeds and up to 16,000 draws a
// row, timed in every form; the predictions are off by 9 to 20% (rms).
struct FormCost {
    int lanes;                    // to a row
    double base;
    double batch, lane_draw;      // of the heaviest row: per batch, and per draw of a lane
    double head;                  // of that, again for every further head of 8,192 rows
    double row, first_rows;       // per 1,000 rows, and of the first 1,000
    double row_batch, draw;       // per 1,000 (row, batch) pairs, per 64,000 draws
    double uneven;                // by how much a Structural row counts as the heaviest, not the mean
    double keys;                  // of the heaviest row: per 65,536 keys of its bitmap
};
double form_us(const MaskParams& p, const RowDraws& d, const FormCost& c) {
    const int most_seeds = c.lanes == 64 ? kSeedBatch<64> : kSeedBatch<256>;
    const double batches = (double)((p.n_seeds + most_seeds - 1) / most_seeds);
    const int64_t pool = p.causal ? p.q0 + p.nq : p.N;
    double domain = 2.0;                                          // a draw's cycle walk: domain / pool steps
    while (domain < (double)pool) domain *= 2.0;
    const double rounds = pool <= 128 ? 2.0 : 1.0;                // twelve rounds to a step instead of six
    const double lane = ceil(p.n_seeds / batches) * d.most / c.lanes;
    const double walk = batches * (c.batch + c.lane_draw * rounds * (domain / (double)pool) * (lane > 1.0 ? lane : 1.0));
    const double heaviest = (d.most > 0.0 ? walk : 0.0) + c.keys * (double)pool / 65536.0;
    const double mean = p.mode == 0 ? d.mean : d.mean + c.uneven * (d.most - d.mean);
    const double rows = 1e-3 * (double)p.heads * (double)p.nq;
    return c.base + heaviest * (1.0 + c.head * (p.heads - 1) * (p.nq < 8192 ? p.nq / 8192.0 : 1.0)) +
           rows * (c.row + c.row_batch * d.share * batches + c.draw * rounds * p.n_seeds * mean / 64.0) +
           c.first_rows * (rows < 1.0 ? rows : 1.0);
}

// One-pass build of light rows: a wave to a row in chunks of 8 or 4, a workgroup to a
// row in chunks of one, or the persistent grid, by the least of the three.  Rows that
// queue are built faster by waves (32,768 rows of one draw 51 us, 300 in the grid);
// few rows, many seeds or heavy rows end with the slowest wave (2,420 rows of 400
// seeds, 40 draws each, 139 us by waves, 81 in the grid; 591 rows of 150 seeds to 59
// draws 69 and 51; 8 heads of 22,781 rows of 70 seeds to 228 draws 3,890 and 3,530),
// and the workgroups are faster than the grid where rows are few (0.6 to 0.9 of its
// time to 2,048 rows).  Of the 6,000 builds 27 are more than 3% slower than in the
// grid with two rows to a ticket; with waves wherever rows are light one in twenty
// was, some by half.
enum class OnePass { kWaves, kChunks, kGrid };
OnePass one_pass_form(const MaskParams& p, const RowDraws& d) {
    const double waves = 0.5 + form_us(p, d, {64, 9.0, 3.6, 0.215, 0.5, 1.8, 0.8, 0.5, 0.125, 0.15, 5.0});
    const double chunks = form_us(p, d, {256, 7.3, 3.05, 0.21, 0.27, 11.4, 8.5, 0.43, 0.064, 0.1, 0.0});
    const double grid = form_us(p, d, {256, 8.7, 3.2, 0.19, 0.0, 12.0, 18.5, 0.15, 0.047, 0.0, 0.0});
    return waves <= chunks && waves <= grid ? OnePass::kWaves : chunks <= grid ? OnePass::kChunks : OnePass::kGrid;
}

// Two-phase build, likewise: 32,768 rows to 2,870 draws 205 us by waves and 290 by
// workgroups, 512 rows of 8,190 draws 31 and 16.  Structural rows count more towards
// their heaviest (31,000 rows of 100 seeds, 31 draws each and 155 at most: 370 and
// 271): of 700 such builds 4 are more than 3% slower than by workgroups alone, 41
// where they count by the mean.  Of all 6,000 count phases 10 are more than 7% slower.
bool two_phase_waves(const MaskParams& p) {
    if (middle_draws(p) >= kWaveDraws || bitmap_words(p) > kWaveKeysTwoPhase / 32) return false;
    const RowDraws d = row_draws(p);
    return 1.0 + form_us(p, d, {64, 4.8, 4.0, 0.12, 0.0, 0.75, 0.0, 0.85, 0.076, 0.2, 1.7}) <=
           form_us(p, d, {256, 4.8, 3.13, 0.187, 0.0, 1.1, 0.0, 2.55, 0.087, 0.0, 0.0});
}

}  // namespace

hipError_t launch_mask_count(const MaskParams& p, int64_t* row_ptr, hipStream_t st) {
    const int64_t rows = (int64_t)p.heads * p.nq;
    if (two_phase_waves(p)) {
        constexpr int kRows = kThreads / 64;
        hipLaunchKernelGGL(k_mask_count<64>, dim3((unsigned)((rows + kRows - 1) / kRows)), dim3(kThreads),
                           group_smem_bytes<64>(p, kRows), st, p, row_ptr);
    } else {
        hipLaunchKernelGGL(k_mask_count<kThreads>, dim3((unsigned)rows), dim3(kThreads), mask_smem_bytes(p), st, p,
                           row_ptr);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_rows, dim3(1), dim3(kScanThreads), 0, st, row_ptr, rows);
    return hipGetLastError();
}

hipError_t launch_mask_fused(const MaskParams& p, int64_t* row_ptr, int32_t* col_idx,
                             int64_t capacity, hipStream_t st) {
    const int64_t rows = (int64_t)p.heads * p.nq, draws = middle_draws(p);
    const RowDraws d = row_draws(p);
    const bool light = draws < kWaveDraws && group_smem_bytes<64>(p, 4) <= kWaveSmem;
    const double batch_draws = d.mean * (p.n_seeds < kSeedBatch<1024> ? p.n_seeds : kSeedBatch<1024>);
    if (rows <= kFewRows && (!light || batch_draws >= kFewRowsDraws))
        return run_mask_chunk<1024, 1>(p, row_ptr, col_idx, capacity, st);
    const OnePass form = light ? one_pass_form(p, d) : OnePass::kGrid;
    if (form == OnePass::kChunks && rows * kThreads <= kMaxItems)
        return run_mask_chunk<kThreads, 1>(p, row_ptr, col_idx, capacity, st);
    if (form == OnePass::kWaves && rows * 64 <= kMaxItems) {
        if (draws < kChunk8Draws && group_smem_bytes<64>(p, 8) <= kChunk8Smem)
            return run_mask_chunk<64, 8>(p, row_ptr, col_idx, capacity, st);
        return run_mask_chunk<64, 4>(p, row_ptr, col_idx, capacity, st);
    }
    hipError_t e = clear_status(row_ptr, rows, rows, 1, st);
    if (e != hipSuccess) return e;
    // Persistent: as many workgroups as fit on the device at once, each
    // taking rows until none is left.
    // Pipeline depth: the deepest (at most 2) that keeps at least 6 workgroups
    // resident per CU; else 0 (each row looks back right after its bitmap).
    int dev = 0, cus = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    int depth = 0, per_cu = 0;
    for (int d = 2; d >= 0; --d) {
        int b = 0;
        e = d == 2 ? fused_occupancy<2>(p, &b) : d == 1 ? fused_occupancy<1>(p, &b) : fused_occupancy<0>(p, &b);
        if (e != hipSuccess) return e;
        if (b >= kMinResidentRows || d == 0) {
            depth = d;
            per_cu = b;
            break;
        }
    }
    int64_t grid = (int64_t)(per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
    if (grid > rows) grid = rows;
    const size_t smem = mask_smem_bytes(p, depth + 1);
    const dim3 g3((unsigned)grid), b3(kThreads);
    if (depth == 2) hipLaunchKernelGGL(k_mask_fused<2>, g3, b3, smem, st, p, row_ptr, col_idx, capacity);
    else if (depth == 1) hipLaunchKernelGGL(k_mask_fused<1>, g3, b3, smem, st, p, row_ptr, col_idx, capacity);
    else hipLaunchKernelGGL(k_mask_fused<0>, g3, b3, smem, st, p, row_ptr, col_idx, capacity);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return strip_status(row_ptr, rows, rows, 1, st);
}

hipError_t launch_mask_fill(const MaskParams& p, const int64_t* row_ptr, int32_t* col_idx,
                            int64_t capacity, hipStream_t st) {
    const int64_t rows = (int64_t)p.heads * p.nq;
    if (two_phase_waves(p)) {
        constexpr int kRows = kThreads / 64;
        hipLaunchKernelGGL(k_mask_fill<64>, dim3((unsigned)((rows + kRows - 1) / kRows)), dim3(kThreads),
                           group_smem_bytes<64>(p, kRows), st, p, row_ptr, col_idx, capacity);
    } else {
        hipLaunchKernelGGL(k_mask_fill<kThreads>, dim3((unsigned)rows), dim3(kThreads), mask_smem_bytes(p), st, p,
                           row_ptr, col_idx, capacity);
    }
    return hipGetLastError();
}

}  // namespace ris
