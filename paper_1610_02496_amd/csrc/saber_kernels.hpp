// Device code of the sparsity-aware LDA sampler for gfx950 (wave64).
// Included once by saber.hip.  Citations refer to the SaberLDA paper.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace saber {

constexpr int kWave = 64;

// ---------------------------------------------------------------------------------------------
// Wavefront primitives (the wave64 counterparts of warp_sum / warp_prefix_sum / warp_vote /
// warp_copy in Sec. 3.2.3): DPP row shifts + row broadcasts for scans, a 64-bit ballot + count
// trailing zeros for the vote, readlane for the copy.
// ---------------------------------------------------------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f32(float v) {
    // lanes without a valid source (or masked rows) receive 0, the identity of the sums below
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_f64(double v) {
    long long b = __double_as_longlong(v);
    int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROW_MASK, 0xf, false);
    int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(uint32_t)lo);
}

// inclusive scan over the 64 lanes: 4 shifts inside each row of 16, then two row broadcasts
#define SABER_SCAN_BODY(T, DPP)                                                            \
    v += DPP<0x111, 0xf>(v); /* row_shr:1 */                                               \
    v += DPP<0x112, 0xf>(v); /* row_shr:2 */                                               \
    v += DPP<0x114, 0xf>(v); /* row_shr:4 */                                               \
    v += DPP<0x118, 0xf>(v); /* row_shr:8 */                                               \
    v += DPP<0x142, 0xa>(v); /* row_bcast:15 into rows 1 and 3 */                          \
    v += DPP<0x143, 0xc>(v); /* row_bcast:31 into rows 2 and 3 */                          \
    return v;
__device__ __forceinline__ float wave_incl_scan(float v) { SABER_SCAN_BODY(float, dpp_f32) }
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) { SABER_SCAN_BODY(uint32_t, dpp_u32) }
__device__ __forceinline__ double wave_incl_scan(double v) { SABER_SCAN_BODY(double, dpp_f64) }
#undef SABER_SCAN_BODY

// binary32 scan used in the sampler's inner loop: the two row-broadcast steps as single fused DPP adds (rows
// outside the row mask keep their value, which is exactly what the scan wants; the compiler fuses a masked DPP
// move into an integer add but not into a float add, hence the two lines of assembly).  s_nop 1 covers the two
// wait states a DPP read needs after the VALU write of its source.  The compiler's hazard recogniser does not see
// inside the assembly, so the one other hazard of a DPP instruction is the caller's to exclude: no VALU write of
// EXEC (v_cmpx, v_readlane into EXEC) within five instructions before the call.  Every call site sits in
// wave-uniform control flow, where EXEC is only ever written by scalar instructions (on gfx9 the compiler forms
// no v_cmpx), which need no wait.
__device__ __forceinline__ float wave_incl_scan_fast(float v) {
    v += dpp_f32<0x111, 0xf>(v);
    v += dpp_f32<0x112, 0xf>(v);
    v += dpp_f32<0x114, 0xf>(v);
    v += dpp_f32<0x118, 0xf>(v);
    asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf" : "+v"(v));
    asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf" : "+v"(v));
    return v;
}

// write a wave-uniform value into one lane of a register
__device__ unsigned int llvm_amdgcn_writelane_u32(unsigned int value, unsigned int lane, unsigned int old)
    __asm("llvm.amdgcn.writelane.i32");

__device__ __forceinline__ float readlane_f32(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ uint32_t readlane_u32(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
    long long b = __double_as_longlong(v);
    int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (long long)(uint32_t)lo);
}
__device__ __forceinline__ float wave_sum(float v) { return readlane_f32(wave_incl_scan(v), 63); }
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return readlane_u32(wave_incl_scan(v), 63); }

// inclusive running maximum over the 64 lanes
__device__ __forceinline__ int wave_incl_scan_max(int v) {
    const int lo = -2147483647 - 1;
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(lo, v, 0x143, 0xc, 0xf, false));
    return v;
}

// index of the first lane whose predicate holds, or -1
__device__ __forceinline__ int wave_vote_first(bool pred) {
    unsigned long long m = __builtin_amdgcn_ballot_w64(pred);
    return m ? (int)__builtin_ctzll(m) : -1;
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Barrier of a workgroup that exchanges data through LDS only: __syncthreads() also waits until every global store in flight
// has been acknowledged by memory, which a kernel that streams its results out does not need between its steps.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11), written for the device; the CPU checker has its own.
// counter = (token lo, token hi, iteration, 0), key = (seed lo, seed hi).
// ---------------------------------------------------------------------------------------------
struct Rand2 { uint32_t r0, r1; };
// Bound by instruction issue: 4.5 cycles for a product of either half or of both, so one v_mad_u64_u32 forms both.  The key is
// opaque at every call: otherwise the compiler computes the 20 round keys once per kernel, has no scalar registers for them,
// and parks them in lanes of a vector register at 4.5 cycles a move, where the scalar unit adds them up for nothing.
__device__ __forceinline__ uint64_t mul_wide(uint32_t a, uint32_t b) {
    uint64_t r;
    asm("v_mad_u64_u32 %0, vcc, %1, %2, 0" : "=v"(r) : "s"(a), "v"(b) : "vcc");
    return r;
}
__device__ __forceinline__ Rand2 philox_token(uint32_t seed_lo, uint32_t seed_hi, uint64_t t, uint32_t iter) {
    uint32_t c0 = (uint32_t)t, c1 = (uint32_t)(t >> 32), c2 = iter, c3 = 0u;
    uint32_t k0 = seed_lo, k1 = seed_hi;
    asm volatile("" : "+s"(k0), "+s"(k1));
#pragma unroll
    for (int r = 0; r < 10; r++) {
        const uint64_t p0 = mul_wide(0xD2511F53u, c0), p1 = mul_wide(0xCD9E8D57u, c2);
        uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ k0, n2 = (uint32_t)(p0 >> 32) ^ c3 ^ k1;
        c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return Rand2{c0, c1};
}
__device__ __forceinline__ float unit24(uint32_t r) { return (float)(r >> 8) * (1.0f / 16777216.0f); }

// ---------------------------------------------------------------------------------------------
// Small utility kernels
// ---------------------------------------------------------------------------------------------
__global__ void fill_u32_kernel(uint32_t *p, uint32_t value, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = value;
}

// z[z_rel + i] belongs to the canonical token t0 + i
template <typename ZT>
__global__ void init_z_kernel(ZT *z, int64_t z_rel, int64_t t0, int64_t t1, uint32_t K, uint32_t seed_lo, uint32_t seed_hi) {
    int64_t t = t0 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (; t < t1; t += stride) {
        Rand2 r = philox_token(seed_lo, seed_hi, (uint64_t)t, 0u);
        z[z_rel + (t - t0)] = (ZT)__umulhi(r.r0, K);   // floor(word0 * K / 2^32)
    }
}

template <typename ZT>
__global__ void z_from_i32_kernel(ZT *z, const int32_t *src, int64_t T) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (; t < T; t += stride) z[t] = (ZT)src[t];
}

// Inspection of a few of a chunk's tokens: marks[t / 32] = {bit t mod 32 set for the tokens t that are asked for, number of the first
// of them among all that are asked for}.  First the bits ...
__global__ void mark_tokens_kernel(const int64_t *idx, int64_t m, int64_t t0, int64_t n, uint2 *marks) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    const int64_t r = idx[i] - t0;
    if (r >= 0 && r < n) atomicOr(&marks[r >> 5].x, 1u << (r & 31));
}
// ... then the numbers: in order inside a workgroup of 256 threads, the workgroups one after the other as they come (*next).
__global__ void __launch_bounds__(256) number_tokens_kernel(uint2 *marks, int64_t words, uint32_t *next) {
    __shared__ uint32_t wave_sum_of[4], base;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t mine = i < words ? (uint32_t)__popc(marks[i].x) : 0u, incl = wave_incl_scan(mine);
    const int wave = threadIdx.x / kWave;
    if (lane_id() == kWave - 1) wave_sum_of[wave] = incl;
    __syncthreads();
    uint32_t before = 0u, all = 0u;
    for (int w = 0; w < 4; w++) { if (w < wave) before += wave_sum_of[w]; all += wave_sum_of[w]; }
    if (threadIdx.x == 0 && all) base = atomicAdd(next, all);
    __syncthreads();
    if (mine) marks[i].y = base + before + (incl - mine);
}
__device__ __forceinline__ bool token_marked(const uint2 m, uint32_t t) { return (m.x >> (t & 31u)) & 1u; }
__device__ __forceinline__ uint32_t token_number(const uint2 m, uint32_t t) { return m.y + (uint32_t)__popc(m.x & ((1u << (t & 31u)) - 1u)); }

// Normalisers of Alg. 2 for the requested tokens that lie in the chunk [t0, t0 + n): S and Q as the sampling
// kernel's inspection mode left them (indexed by the token's position in the chunk, or by its number among the marked ones) and
// the probability of the sparse branch, S / (S + Q).
__global__ void gather_probs_kernel(const float *S, const float *Q, const uint2 *marks, const int64_t *idx, int64_t m, int64_t t0, int64_t n,
                                    float *out_S, float *out_Q, float *out_p) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    int64_t r = idx[i] - t0;
    if (r < 0 || r >= n) return;
    if (marks) r = token_number(marks[r >> 5], (uint32_t)(r & 31));
    const float s = S[r], q = Q[r];
    out_S[i] = s; out_Q[i] = q; out_p[i] = s / (s + q);
}

// ---------------------------------------------------------------------------------------------
// Work description of the E-step: one tile = up to tile_tokens tokens of one word inside one chunk.
// Tokens of a chunk are stored word-major (partition-by-document, order-by-word, Sec. 3.1.4).
// ---------------------------------------------------------------------------------------------
// row: the word's row in the dense B / Bhat arrays, or its index among the light words (see below)
// wm_begin: position of the tile's first token in the corpus-wide word-major order
// range: host only, 1 + range of documents the tile was cut to (0: whole)
struct Tile { int32_t word; int32_t begin; int32_t count; int32_t row; int64_t wm_begin; int64_t range; };

struct EStepParams {
    const Tile *tiles;
    const int32_t *tok_doc;     // [chunk tokens] document of the token (global document id)
    const uint32_t *tok_t;      // [chunk tokens] canonical token index relative to t_base
    const uint2 *docrec;        // [D] {row start in units of 32 entries, K_d}
    const uint32_t *cd_rows;    // packed rows of A (count | topic << count_bits, ascending topic) from the first row of
                                // the chunk's documents on: the row of document d starts (docrec[d].x - row_unit0) * 32
                                // entries into it
    uint32_t row_unit0;         // row start of the chunk's first document
    uint32_t rows_bytes;        // bytes from cd_rows to the end of the chunk's last row (below 2^32)
    uint32_t quarter_row_bytes; // rows up to this padded length (at most 256 bytes) are sampled four at a time, one per 16 lanes
    uint32_t half_row_bytes;    // longer rows up to this length (at most 512 bytes) two at a time, one per 32 lanes
    const float *phi;           // [dense rows][Kpad]  Bhat
    const float *l3;            // [V][n3pad] binary32 prefix sum of the Bhat row at the end of every 64-topic block,
                                //            padded with the row total (tree level above the bottom)
    const double *l3_64;        // [V][n3]    the same running sums before rounding (base of each bottom block)
    const float *sumphi;        // [V]        prefix sum at topic K-1 = l3[n3-1]
    void *z;                    // assignments in canonical order (uint16 or int32): the chunk's token t_base + i is
                                // element z_rel + i (the resident array holds all tokens, a streaming buffer one chunk)
    // light words (few tokens): B is kept sparse, Bhat = base + the word's non-zeros
    const float *base;          // [Kpad] Bhat of a zero count, beta / denom_k (pad columns 0)
    const uint2 *wrec;          // [light words] {row start in units of 32 entries, non-zeros}
    const uint32_t *lw_ent;     // packed (topic, count) rows of B for the light words, ascending topic
    const float *lw_phi;        // Bhat value of every such entry
    void *z_wm;                 // [T] new assignments in word-major order (light words first): input of CountByVZ
    const uint2 *alias_table;   // null, or [dense rows][K] {prob bits, alias}: the dense term is then drawn from these
                                // alias tables instead of the prefix-sum tree (measurement variant, Sec. 3.2.3)
    const uint2 *marks;         // probs mode: null, or the only tokens that S and Q are asked for (mark_tokens_kernel)
    float *out_S;               // probs mode: S per token of the chunk, indexed by its position in the chunk or its number among the marked
    float *out_Q;               // probs mode: Q likewise
    double *out_ll;             // loglik mode: one partial sum per tile
    unsigned long long *n_dense;// sample mode: kDenseSlots dense-branch token counters (workgroup b adds to slot b mod
                                // kDenseSlots: one hot address would serialise the atomics of the whole launch)
    int32_t first_light;        // tiles of the launch from this one on belong to light words
    int32_t n_tiles, walkers;   // tiles of the launch; workgroups its light words' tiles are dealt to: each works on every walkers-th
    int64_t t_base;             // canonical index of the chunk's first token
    int64_t z_rel;              // position of that token in z
    int32_t K, Kpad, n3, n3pad;
    uint32_t count_bits;        // low bits of an entry that hold its count
    float alpha;
    uint32_t seed_lo, seed_hi, iter;
};

enum { MODE_SAMPLE = 0, MODE_PROBS = 1, MODE_LOGLIK = 2 };
constexpr int kDenseSlots = 1024;

// Sums and scans inside one DPP row (16 lanes): the dense branch serves four tokens at a time, one per row.
__device__ __forceinline__ uint32_t row16_allsum(uint32_t v) {
    v += dpp_u32<0x128, 0xf>(v);   // row_ror:8
    v += dpp_u32<0x124, 0xf>(v);   // row_ror:4
    v += dpp_u32<0x122, 0xf>(v);   // row_ror:2
    v += dpp_u32<0x121, 0xf>(v);   // row_ror:1
    return v;
}
__device__ __forceinline__ double row16_incl_scan(double v) {
    v += dpp_f64<0x111, 0xf>(v);
    v += dpp_f64<0x112, 0xf>(v);
    v += dpp_f64<0x114, 0xf>(v);
    v += dpp_f64<0x118, 0xf>(v);
    return v;
}

__device__ __forceinline__ float row16_incl_scan(float v) {
    v += dpp_f32<0x111, 0xf>(v);
    v += dpp_f32<0x112, 0xf>(v);
    v += dpp_f32<0x114, 0xf>(v);
    v += dpp_f32<0x118, 0xf>(v);
    return v;
}

// A light word's Bhat row where LDS cannot hold one: the base vector in memory, and for each of the word's non-zeros a mark in
// LDS, marks[k / 32] = {bit k mod 32 set where topic k has a count, number of the non-zeros before the first of these}, which
// leads to its value.  light: wave-uniform; without it the row is read as it is.
struct Overlay { const uint2 *marks = nullptr; const float *val = nullptr; bool light = false; };

// Dense branch (problem 2, Sec. 2.3): position of x in the prefix sums of the word's Bhat row, four tokens per
// call: the 16 lanes of DPP row g serve the token whose x they hold (all lanes of a row hold the same x).
// The descent follows Sec. 3.2.4 with the stored level l3 (binary32 prefix sum at the end of every 64-topic
// block; every 16th, 256th, ... entry of it acts as the levels above).  Prefix sums are non-decreasing, so
// "first entry >= x" is the number of entries below x: every lane tests one entry and one row-wide sum gives
// the position.  The bottom level is not stored: the 64 prefix sums of the chosen block are rebuilt from the
// Bhat values as round32(base + running sum in binary64), base = unrounded running sum at the block's start -
// the numbers a stored table would hold, so the search is exact.
// Those 64 numbers are first formed in binary32 alone (base = the stored, rounded running sum before the block):
// 12 roundings of positive numbers put each within 7.5e-7 of the exact one, relatively.  If none of them lies within
// 1.5e-6 x of x, the count of entries below x is the same for both and the binary64 arithmetic (and the load of its
// base) is skipped; otherwise (a few calls in a hundred at K = 10,000) the exact numbers decide.
// Returns the topic in every lane of the row.
__device__ __forceinline__ uint32_t dense_query4(const float *phi_row, int phi_len, const float *l3,
                                                 const double *__restrict__ l3_64, int n3, int K, float x, int li, const Overlay &ov = Overlay()) {
    // 16-ary descent over l3: lane li looks at the last entry of the li-th sub-range of the current window; the
    // number of sub-ranges lying wholly below x is the index of the one holding the position
    int stride = 1;
    while (stride * 16 < n3) stride *= 16;
    int blk = 0;
    for (; stride >= 1; stride >>= 4) {
        const float c = l3[min(blk + (li + 1) * stride - 1, n3 - 1)];
        blk += min((int)row16_allsum(c < x ? 1u : 0u), 15) * stride;
    }
    blk = min(blk, n3 - 1);                                 // rounding left no block: the last one
    const int k0 = blk * kWave + li * 4;
    float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k0 < phi_len) f = *reinterpret_cast<const float4 *>(phi_row + k0);   // columns K..phi_len-1 hold zeros
    if (ov.light && k0 < K) {                               // four topics of one word of the bitmap
        const uint2 m = ov.marks[k0 >> 5];
        const uint32_t sh = (uint32_t)k0 & 31u, four = (m.x >> sh) & 15u;
        const float *v = ov.val + m.y + __popc(m.x & ((1u << sh) - 1u));
        if (four & 1u) f.x = *v++;
        if (four & 2u) f.y = *v++;
        if (four & 4u) f.z = *v++;
        if (four & 8u) f.w = *v;
    }
    const float t0 = f.x, t1 = t0 + f.y, t2 = t1 + f.z, t3 = t2 + f.w;
    const float a2 = (blk > 0 ? l3[blk - 1] : 0.f) + (row16_incl_scan(t3) - t3);
    const float c0 = a2 + t0, c1 = a2 + t1, c2 = a2 + t2, c3 = a2 + t3;
    uint32_t below = (c0 < x ? 1u : 0u) + (c1 < x ? 1u : 0u) + (c2 < x ? 1u : 0u) + (c3 < x ? 1u : 0u);
    const float nearest = fminf(fminf(fabsf(c0 - x), fabsf(c1 - x)), fminf(fabsf(c2 - x), fabsf(c3 - x)));
    if (__builtin_amdgcn_ballot_w64(nearest <= x * 1.5e-6f)) {   // wave-uniform: some entry is too close to x to call
        const double base = blk > 0 ? l3_64[blk - 1] : 0.0;
        const double s0 = (double)f.x, s1 = s0 + (double)f.y, s2 = s1 + (double)f.z, s3 = s2 + (double)f.w;
        const double b2 = base + (row16_incl_scan(s3) - s3);
        below = ((float)(b2 + s0) < x ? 1u : 0u) + ((float)(b2 + s1) < x ? 1u : 0u) +
                ((float)(b2 + s2) < x ? 1u : 0u) + ((float)(b2 + s3) < x ? 1u : 0u);
    }
    const int k = blk * kWave + min((int)row16_allsum(below), kWave - 1);
    return (uint32_t)min(k, K - 1);
}

// How many of the 16 lanes of this lane's DPP row satisfy pred (row_shift = 16 * row): one compare into a
// wave-wide mask, the row's 16 bits of it, a bit count.
__device__ __forceinline__ uint32_t row16_count(bool pred, uint32_t row_shift) {
    const unsigned long long m = __builtin_amdgcn_ballot_w64(pred);
    return (uint32_t)__builtin_popcount((uint32_t)(m >> row_shift) & 0xffffu);
}

// dense_query4 for a workgroup that holds the word's Bhat row and tree level in LDS, laid out as the sampling
// kernel stages them: the row from byte 0 to phi_bytes (K rounded to 4 floats), four control words of which the
// last is zero, then l3 from byte l3_addr = phi_bytes + 16.  Same numbers and same decisions as dense_query4; what
// differs is how they are fetched and counted.  Nothing is read conditionally: l3[-1] is the zero word before l3[0];
// a lane whose four columns lie past the row's end (last block only) reads the row's last four instead and is left
// out of the count afterwards (its sums would not be below x, and a prefix scan hands nothing of it to the lanes
// before it).  The descent's strides are powers of 16, applied as shifts (top_shift = 4 * number of levels above
// the lowest), and a row's count of entries below x comes from one wave-wide compare mask instead of four DPP additions.
__device__ __forceinline__ uint32_t dense_query4_staged(uint32_t phi_bytes, uint32_t l3_addr, const double *__restrict__ l3_64,
                                                        int n3, int top_shift, int K, float x, uint32_t li, uint32_t row_shift) {
    typedef __attribute__((address_space(3))) const float lds_cfloat;
    typedef float quad_t __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const quad_t lds_cquad;
    uint32_t blk = 0;
    for (int sh = top_shift; sh >= 0; sh -= 4) {
        const uint32_t probe = min(blk + ((li + 1u) << sh), (uint32_t)n3);   // 1 + index of the entry this lane tests
        const float c = *reinterpret_cast<lds_cfloat *>(l3_addr - 4u + (probe << 2));
        blk += min(row16_count(c < x, row_shift), 15u) << sh;
    }
    blk = min(blk, (uint32_t)n3 - 1u);                      // rounding left no block: the last one
    const uint32_t col_bytes = (blk << 8) + (li << 4);
    const bool in_row = col_bytes < phi_bytes;
    const quad_t f = *reinterpret_cast<lds_cquad *>(min(col_bytes, phi_bytes - 16u));
    const float before = *reinterpret_cast<lds_cfloat *>(l3_addr - 4u + (blk << 2));
    const float t0 = f.x, t1 = t0 + f.y, t2 = t1 + f.z, t3 = t2 + f.w;
    const float a2 = before + (row16_incl_scan(t3) - t3);
    const float c0 = a2 + t0, c1 = a2 + t1, c2 = a2 + t2, c3 = a2 + t3;
    uint32_t below = (c0 < x ? 1u : 0u) + (c1 < x ? 1u : 0u) + (c2 < x ? 1u : 0u) + (c3 < x ? 1u : 0u);
    const float nearest = fminf(fminf(fabsf(c0 - x), fabsf(c1 - x)), fminf(fabsf(c2 - x), fabsf(c3 - x)));
    if (__builtin_amdgcn_ballot_w64(in_row && nearest <= x * 1.5e-6f)) {   // wave-uniform: some entry is too close to x to call
        const double base = blk > 0 ? l3_64[blk - 1] : 0.0;
        const double s0 = (double)f.x, s1 = s0 + (double)f.y, s2 = s1 + (double)f.z, s3 = s2 + (double)f.w;
        const double b2 = base + (row16_incl_scan(s3) - s3);
        below = ((float)(b2 + s0) < x ? 1u : 0u) + ((float)(b2 + s1) < x ? 1u : 0u) +
                ((float)(b2 + s2) < x ? 1u : 0u) + ((float)(b2 + s3) < x ? 1u : 0u);
    }
    const uint32_t k = (blk << 6) + min(row16_allsum(in_row ? below : 0u), (uint32_t)kWave - 1u);
    return min(k, (uint32_t)K - 1u);
}

// ---------------------------------------------------------------------------------------------
// E-step (Alg. 2).  One workgroup per tile, or per several tiles of light words where rows are long; the word's Bhat row and the upper tree level are staged in
// LDS (STAGED) or read from global memory.  Each wavefront takes a batch of up to 64 tokens: the
// per-token scalars (document, row descriptor, Philox draws) are produced one token per lane.  Tokens are
// ordered by (word, document), so repeated occurrences of a word in a document are neighbours (a "run"): they
// share A_d (.) Bhat_v and S, and only the two draws differ.
//
// A row of A is consumed in pieces of 4 entries per lane (one 16-byte load per lane): the lane forms its four
// running partial products, a DPP scan over the lane sums yields both S and every prefix sum, and the draw is
// located with one ballot plus a four-way compare inside the winning lane.  How many lanes a run gets depends
// on the length of its row:
//   * rows of at most 64 entries: four runs at a time, one per DPP row of 16 lanes;
//   * rows of at most 128 entries: two runs at a time, one per half of the wavefront;
//   * longer rows: one run at a time over all 64 lanes, in blocks of 256 entries.
// A lane's 16 entries sit in the same order in all three layouts and a DPP scan never crosses the lanes of a
// group, so the sums come out bit-identical whichever layout a row gets.
// PACK: how an entry holds its topic (in the high bits) and its count (in the low ones).
// ---------------------------------------------------------------------------------------------
enum {
    PACK_ANY = 0,     // count_bits is a run-time value
    PACK_16 = 1,      // 16 bits each
    PACK_16_14 = 2,   // 16 bits each, and all counts below 2^14: the entry shifted down by 14 is then the topic times 4
};

struct RowBlock { float a0, a1, a2, a3, incl; };   // running sums inside the lane; inclusive scan of lane sums

// One 256-entry block of a row: lane l receives entries 4l..4l+3 through a buffer load whose descriptor ends
// at the row's padded length, so lanes past the end read zeros without any branch.  Rows are 128-byte
// aligned and padded to a multiple of 4 entries with (last topic, count 0).
__device__ __forceinline__ uint4 load_block(const uint32_t *row, int rel_kd, int lane) {
    const int bytes = rel_kd > 0 ? ((rel_kd + 3) & ~3) * 4 : 0;
    __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)row, (short)0, bytes, 0x00020000);
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane * 16, 0, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// 16 bytes at a per-lane byte offset into the rows of a chunk; an offset of 0xffffffff (any offset past the
// descriptor's end) returns zeros and moves no data.
__device__ __forceinline__ uint4 load_rows_at(__amdgpu_buffer_rsrc_t rows, uint32_t byte_off) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rows, (int)byte_off, 0, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// clear bit `bit` of a wave-uniform mask (one scalar instruction)
__device__ __forceinline__ unsigned long long clear_bit(unsigned long long m, int bit) {
    asm("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(bit));
    return m;
}

// lowest set bit of a wave-uniform mask, -1 if there is none
__device__ __forceinline__ int first_bit(unsigned long long m) {
    int i;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(i) : "s"(m));
    return i;
}

// What a wavefront wrote to its own part of LDS is in LDS order before what it reads there next; this keeps the compiler to it.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// lane permutations through the LDS crossbar (no LDS memory is touched); lane numbers are passed times 4
__device__ __forceinline__ uint32_t lane_pull(uint32_t v, uint32_t src_lane4) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)src_lane4, (int)v);      // every lane reads lane src
}
__device__ __forceinline__ float lane_pull(float v, uint32_t src_lane4) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute((int)src_lane4, __float_as_int(v)));
}
__device__ __forceinline__ uint32_t lane_push(uint32_t v, uint32_t dst_lane4) {
    return (uint32_t)__builtin_amdgcn_ds_permute((int)dst_lane4, (int)v);       // every lane writes lane dst; the
}                                                                               // highest writer wins, unwritten lanes get 0

// lane 31's value in lanes 0 to 31, lane 63's in the others (a fixed pattern takes 2.3 cycles of a CU's LDS, a pull 6.1)
__device__ __forceinline__ float half_last(float v) {
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), 31 << 5));
}

// number of set bits of a wave-uniform mask at this lane or below it
__device__ __forceinline__ uint32_t bits_up_to_lane(unsigned long long m) {
    const unsigned long long h = m >> 1;
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(h >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h, (uint32_t)(m & 1ull)));
}

// Inclusive scan over the lanes of each group of G lanes (G = 16: one DPP row; 32: half a wavefront; 64: all).
template <int G>
__device__ __forceinline__ float group_incl_scan(float v) {
    v += dpp_f32<0x111, 0xf>(v);
    v += dpp_f32<0x112, 0xf>(v);
    v += dpp_f32<0x114, 0xf>(v);
    v += dpp_f32<0x118, 0xf>(v);
    // see wave_incl_scan_fast for the two lines of assembly and their precondition
    if (G >= 32) asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf" : "+v"(v));
    if (G >= 64) asm volatile("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf" : "+v"(v));
    return v;
}

// Bhat value of the entry's topic.  With 16/16 packing and the row in LDS the byte offset (topic * 4) is formed by one shift: of the
// entry where nothing of the count gets into it, otherwise one that reads the entry's high half (4.5 cycles of the vector unit
// against 2.5).
template <bool STAGED, int PACK>
__device__ __forceinline__ float phi_of(uint32_t e, uint32_t cbits, const float *lds_phi, const float *__restrict__ phi_row, const Overlay &ov) {
    if (STAGED && PACK != PACK_ANY) {
        uint32_t off;
        if (PACK == PACK_16_14) off = e >> 14;
        else asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
                 : "=v"(off) : "v"(2u), "v"(e));
        // the staged row starts at LDS address 0 (the kernel has no static LDS; the host checks that at start-up)
        typedef __attribute__((address_space(3))) const float lds_cfloat;
        return *reinterpret_cast<lds_cfloat *>(off);
    }
    const uint32_t k = e >> cbits;
    if (STAGED) return lds_phi[k];
    const float *src = phi_row + k;
    if (ov.light) {   // the value is where the mark says: one load either way
        const uint2 m = ov.marks[k >> 5];
        const uint32_t below = (1u << (k & 31u)) - 1u;
        if ((m.x >> (k & 31u)) & 1u) src = ov.val + (m.y + __popc(m.x & below));
    }
    return *src;
}

// element-wise product A_d (.) Bhat_v of the lane's four entries as running sums, and their scan over the group
template <bool STAGED, int PACK, int G = kWave>
__device__ __forceinline__ void block_products(const uint4 e, uint32_t cbits, const float *lds_phi, const float *__restrict__ phi_row,
                                               RowBlock &b, const Overlay &ov = Overlay()) {
    const float f0 = phi_of<STAGED, PACK>(e.x, cbits, lds_phi, phi_row, ov);
    const float f1 = phi_of<STAGED, PACK>(e.y, cbits, lds_phi, phi_row, ov);
    const float f2 = phi_of<STAGED, PACK>(e.z, cbits, lds_phi, phi_row, ov);
    const float f3 = phi_of<STAGED, PACK>(e.w, cbits, lds_phi, phi_row, ov);
    const uint32_t cmask = PACK != PACK_ANY ? 0xffffu : (1u << cbits) - 1u;
    b.a0 = (float)(e.x & cmask) * f0;
    b.a1 = __builtin_fmaf((float)(e.y & cmask), f1, b.a0);
    b.a2 = __builtin_fmaf((float)(e.z & cmask), f2, b.a1);
    b.a3 = __builtin_fmaf((float)(e.w & cmask), f3, b.a2);
    b.incl = group_incl_scan<G>(b.a3);
}

// First entry of the block whose prefix sum (carry + sums inside the block) reaches x.  The lane is found
// with one ballot over the lanes' inclusive sums, the entry inside it with three compares.  If rounding
// leaves no entry, the choice falls on the block's last one (a row's padding repeats its last topic).  Returns the entry.
__device__ __forceinline__ uint32_t search_block(const uint4 e, const RowBlock &b, float carry, float x, int rel_kd) {
    const float base = carry + (b.incl - b.a3);
    const unsigned long long m3 = __builtin_amdgcn_ballot_w64(carry + b.incl >= x);
    const int nvalid = rel_kd < 4 * kWave ? rel_kd : 4 * kWave;
    const int L = m3 ? (int)__builtin_ctzll(m3) : ((nvalid - 1) >> 2);
    uint32_t sel = e.w;
    sel = base + b.a2 >= x ? e.z : sel;
    sel = base + b.a1 >= x ? e.y : sel;
    sel = base + b.a0 >= x ? e.x : sel;
    return readlane_u32(sel, L);
}

// The kernel's parameters where the hardware left them, read again from there (constant memory, scalar loads).  The compiler reads
// them once, at the top, and has no scalar registers for what the batch loop needs only now and then: it parked 64 of them in
// the lanes of a vector register, and moved them there and back at 4.5 cycles of the vector unit each, 64 moves when a wavefront
// starts and 80 per batch.  With the round keys of philox_token out of them too: T = 10 M, K = 1,000 an iteration of 654 -> 643
// us, T = 15 M, K = 20,011 2,000 -> 1,977, T = 100 M, K = 10,000 7,618 -> 7,585.
typedef __attribute__((address_space(4))) const EStepParams EStepParamsConst;
__device__ __forceinline__ EStepParamsConst *params_again() {
    auto *q = (EStepParamsConst *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));   // (a pointer the compiler knows nothing of: nothing read through it earlier is kept)
    return q;
}

__device__ __forceinline__ float first_lane(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

// What a kernel only reads, read with the scalar unit where the address is the same for a whole wavefront (behind a store the
// compiler takes the vector unit: the store might have changed it).
template <typename T> using ConstMem = __attribute__((address_space(4))) const T;
template <typename T> __device__ __forceinline__ ConstMem<T> *const_mem(const T *p) { return (ConstMem<T> *)(uintptr_t)p; }

// New assignments are written twice: to z (canonical order) and to z_wm (word-major, coalesced), from which the
// M-step counts B; the sampler itself adds nothing to B.
// A light word keeps B sparse: its Bhat row is built in LDS from the base vector and the word's non-zeros (staged rows have
// 16-bit assignments then), or where LDS cannot hold a row read from memory with marks in LDS (Overlay).  Tiles of both kinds share a launch: a launch of its own for the light words cost a small
// corpus 10 of its 47 us per iteration (T = 100 K, K = 100), a large one the tail of the other.
// Tokens of a run from which on their positions in its row are looked for at once (5 to 9; a fifth of the tokens are in runs of 16
// and more, 28 per cent in runs of 8 and more).  One token after the other takes ten vector and six scalar instructions each, all
// of a run's at once about 35 and 13 lane permutations.  An iteration at T = 100 M, K = 10,000 7.34 -> 7.21 ms, T = 10 M, K = 1,000
// 575 -> 562 us; from 6 or 12 tokens on the same within 0.5 %.
constexpr int kManyTokens = 8;
// SLOTS (sampling): a wavefront has kSlotBytes of LDS of its own, through which short rows' runs and their tokens exchange what
// they need, instead of lane permutations.
constexpr int kSpareSlots = 8;                                             // read ahead by the last passes
constexpr uint32_t kSlotBytes = kWave * 4 + (kWave + kSpareSlots) * 8;     // a word per token, then a pair per piece of a run
template <int MODE, bool STAGED, typename ZT, int PACK, bool SLOTS = false>
__global__ void __launch_bounds__(1024, 8) estep_kernel(EStepParams p) {
    extern __shared__ float4 lds_f4[];
    // LDS, all of it dynamic so that the Bhat row starts at address 0 and a gather needs no base added:
    //   STAGED: [K rounded to 4] floats: the word's Bhat row
    //   [4] words: batch ticket, dense-branch tokens of the workgroup, whether a token is asked for (probs mode), 0 (the tree
    //           level's entry "before the first", which the dense branch reads for the first block)
    //   STAGED: [n3 rounded to 4] floats: the tree level above the bottom;  LOGLIK: [16] doubles, one per wavefront
    //   SLOTS: kSlotBytes per wavefront
    //   not STAGED, if some words are light: after room for these 16 doubles, a pair of words per 32 topics (Overlay)
    // The footprint is kept minimal because it decides how many wavefronts a CU can hold: at K = 10,000 it is
    // 40,656 bytes, which lets four 512-thread workgroups (32 wavefronts) share the 160 KB of a CU.
    const int K4 = STAGED ? (p.K + 3) & ~3 : 0;
    float *lds_phi = reinterpret_cast<float *>(lds_f4);
    int *ctrl = reinterpret_cast<int *>(lds_phi + K4);
    float *lds_l3 = lds_phi + K4 + 4;
    double *ll_wave = reinterpret_cast<double *>(lds_l3 + (STAGED ? (p.n3 + 3) & ~3 : 0));
    constexpr bool kWalks = STAGED && sizeof(ZT) == 2 && MODE == MODE_SAMPLE;   // (see walkers_for() on the host)
    int tile_at = (int)blockIdx.x;
    const Tile tile = p.tiles[tile_at];
    const bool light = (!STAGED || sizeof(ZT) == 2) && (int)blockIdx.x >= p.first_light;
    const int K = p.K;
    if (MODE == MODE_PROBS && p.marks) {   // nothing to do, and no row to stage, where none of the tile's tokens is asked for
        if (threadIdx.x == 0) ctrl[2] = 0;
        __syncthreads();
        bool any = false;
        for (int i = threadIdx.x; i < tile.count; i += blockDim.x) {
            const uint32_t tt = p.tok_t[tile.begin + i];
            any |= token_marked(p.marks[tt >> 5], tt);
        }
        if (any) ctrl[2] = 1;
        __syncthreads();
        if (ctrl[2] == 0) return;
    }
    const float *__restrict__ phi_row = light ? p.base : p.phi + (size_t)tile.row * (size_t)p.Kpad;
    const float *__restrict__ l3_row = p.l3 + (size_t)tile.word * (size_t)p.n3pad;
    int lane = lane_id();
    const int nwaves = blockDim.x / kWave;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    // batch size: 64 tokens per wavefront, fewer when the tile is too small to keep every wavefront busy
    int bs = (tile.count + nwaves - 1) / nwaves;
    bs = __builtin_amdgcn_readfirstlane(bs > kWave ? kWave : bs);   // wave-uniform: keep it in a scalar register
    // The first batch of every wavefront is fixed (wavefront w takes batch w; the ticket counter starts behind these),
    // so its token records are requested here, before the word's row is staged, and the row records of their
    // documents before the workgroup waits at the barrier: for a small tile (one batch per wavefront) two of the three
    // dependent memory accesses in front of the first row then pass under the staging.
    int batch = wave * bs;
    int d = -1;
    uint32_t t = 0u;
    if (lane < min(bs, tile.count - batch)) {
        d = p.tok_doc[tile.begin + batch + lane];
        t = p.tok_t[tile.begin + batch + lane];
    }
    if (threadIdx.x == 0) { ctrl[0] = nwaves; ctrl[1] = 0; ctrl[3] = 0; }
    auto stage_row = [&](const int tid, const float *src, const int K4) {
        // eight 16-byte loads per thread are requested before the first of them is written to LDS: one load, one
        // wait, one write at a time left a workgroup's start waiting for memory five times over at K = 10,000.
        // (No branch inside: past the end, the last piece is read and written once more.)
        typedef float quad_t __attribute__((ext_vector_type(4)));
        const quad_t *qsrc = reinterpret_cast<const quad_t *>(src);
        quad_t *qdst = reinterpret_cast<quad_t *>(lds_phi);
        const int nq = K4 / 4, step = (int)blockDim.x;
        for (int i0 = tid; i0 < nq; i0 += 8 * step) {
            const quad_t q0 = qsrc[min(i0, nq - 1)], q1 = qsrc[min(i0 + step, nq - 1)], q2 = qsrc[min(i0 + 2 * step, nq - 1)],
                         q3 = qsrc[min(i0 + 3 * step, nq - 1)], q4 = qsrc[min(i0 + 4 * step, nq - 1)],
                         q5 = qsrc[min(i0 + 5 * step, nq - 1)], q6 = qsrc[min(i0 + 6 * step, nq - 1)],
                         q7 = qsrc[min(i0 + 7 * step, nq - 1)];
            qdst[min(i0, nq - 1)] = q0; qdst[min(i0 + step, nq - 1)] = q1; qdst[min(i0 + 2 * step, nq - 1)] = q2;
            qdst[min(i0 + 3 * step, nq - 1)] = q3; qdst[min(i0 + 4 * step, nq - 1)] = q4; qdst[min(i0 + 5 * step, nq - 1)] = q5;
            qdst[min(i0 + 6 * step, nq - 1)] = q6; qdst[min(i0 + 7 * step, nq - 1)] = q7;
        }
    };
    if (STAGED) {
        stage_row((int)threadIdx.x, phi_row, K4);
        if (MODE == MODE_SAMPLE)
            for (int i = threadIdx.x; i < p.n3; i += blockDim.x) lds_l3[i] = l3_row[i];
    }
    uint2 rec = make_uint2(p.row_unit0, 0u);
    if (d >= 0) rec = p.docrec[d];
    Overlay ov;
    if (!STAGED && light) {
        uint2 *marks = reinterpret_cast<uint2 *>(lds_l3 + 32);
        const uint2 wr = p.wrec[tile.row];
        const uint32_t *__restrict__ ent = p.lw_ent + (size_t)wr.x * 32u;
        for (int i = threadIdx.x; i < (K + 31) >> 5; i += blockDim.x) marks[i].x = 0u;
        __syncthreads();
        for (int j = threadIdx.x; j < (int)wr.y; j += blockDim.x) {   // (ascending topics)
            const uint32_t k = ent[j] >> p.count_bits, before = j ? ent[j - 1] >> p.count_bits : 0xffffffffu;
            atomicOr(&marks[k >> 5].x, 1u << (k & 31u));
            if (before >> 5 != k >> 5) marks[k >> 5].y = (uint32_t)j;
        }
        ov = Overlay{marks, p.lw_phi + (size_t)wr.x * 32u, true};
    }
    if (STAGED && light) {
        // the staged row is the base vector so far; overwrite the topics this word has counts for.  The word's first
        // entries, one per thread, are requested before the barrier as well: with few tokens per workgroup the chain of
        // dependent loads shows (T = 15 M, K = 20,011, 76 tokens per light word: pass 1.920 -> 1.829 ms; elsewhere within 0.5 %).
        const uint2 wr = p.wrec[tile.row];
        const uint32_t *__restrict__ ent = p.lw_ent + (size_t)wr.x * 32u;
        const float *__restrict__ val = p.lw_phi + (size_t)wr.x * 32u;
        const uint32_t cb = PACK != PACK_ANY ? 16u : p.count_bits;
        uint32_t e0 = 0u; float v0 = 0.f;
        if ((int)threadIdx.x < (int)wr.y) { e0 = ent[threadIdx.x]; v0 = val[threadIdx.x]; }
        __syncthreads();
        if ((int)threadIdx.x < (int)wr.y) lds_phi[e0 >> cb] = v0;
        for (int j = threadIdx.x + blockDim.x; j < (int)wr.y; j += blockDim.x) lds_phi[ent[j] >> cb] = val[j];
    }
    __syncthreads();
    float sum_w = *const_mem(p.sumphi + tile.word);
    float Q = first_lane(p.alpha * sum_w);
    const uint32_t cbits = PACK != PACK_ANY ? 16u : p.count_bits;
    int count = tile.count;
    // The tiles of the workgroup.  More than one, and then of light words, is for sampling from staged rows with 16-bit assignments:
    // bound by the chain from a tile's record to its rows of A, and by staging a row per tile before that (80 KB at K = 20,011:
    // 2.03 -> 1.67 ms per iteration at T = 15 M).
    for (;;) {
    asm volatile("" : "+v"(lane));   // (values derived from the lane number are formed per tile, not held over all of them)
    double ll_acc = 0.0;
    // `batch`, and d, t, rec of its tokens, are in hand at the top of every turn: those of the first batch from above,
    // those of the later ones from the bottom of the turn before
    if (batch < count)
    for (int round = 0;; round++) {
        const int n = __builtin_amdgcn_readfirstlane(min(bs, count - batch));   // wave-uniform by construction
        bool act = lane < n;
        if (MODE == MODE_PROBS && p.marks && act) act = token_marked(p.marks[t >> 5], t);   // each of them a run of its own
        float u0 = 0.f, u1 = 0.f;
        EStepParamsConst *q = params_again();
        const uint32_t row_unit0 = q->row_unit0;
        // all rows of A of the chunk behind one buffer descriptor: a row is addressed by its 32-bit byte offset
        const char *rows_base = reinterpret_cast<const char *>(q->cd_rows);
        const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(rows_base), (short)0, (int)q->rows_bytes, 0x00020000);
        if (MODE == MODE_SAMPLE) {
            Rand2 r = philox_token(q->seed_lo, q->seed_hi, (uint64_t)(q->t_base + (int64_t)t), q->iter);
            u0 = unit24(r.r0); u1 = unit24(r.r1);
        }
        uint32_t my_z = 0; float my_S = 0.f;
        unsigned long long sparse_mask = 0ull;   // tokens that take the sparse branch

        // Runs: bit i of `starts` marks a lane where the tokens of another document begin.
        const int d_prev = __builtin_amdgcn_update_dpp(-2, d, 0x138, 0xf, 0xf, false);   // wave_shr:1
        // (masks of the active lanes by a scalar AND: a compare of both at once goes by way of a vector register)
        const unsigned long long acts = __builtin_amdgcn_ballot_w64(act);
        const bool alone = MODE == MODE_PROBS && p.marks;
        const unsigned long long starts = ((alone ? ~0ull : __builtin_amdgcn_ballot_w64(d != d_prev)) & acts) | (alone ? 0ull : 1ull);
        // the row of the lane's document: byte offset inside the chunk's rows and padded length in bytes
        const uint32_t row_off = (rec.x - row_unit0) << 7;
        const uint32_t row_bytes = ((rec.y + 3u) & ~3u) << 2;
        const int row_last = (int)(row_bytes >> 4) - 1;   // number of its last piece of 16 bytes
        // position of the token inside its run
        const uint32_t jpos = (uint32_t)(lane - wave_incl_scan_max(__builtin_amdgcn_inverse_ballot_w64(starts | 1ull) ? lane : -1));
        // rows that fit a quarter or a half of the wavefront; runs are cut into pieces of at most G tokens there
        const uint32_t quarter = q->quarter_row_bytes, half = q->half_row_bytes;
        unsigned long long m16 = __builtin_amdgcn_ballot_w64(row_bytes <= quarter) & acts;
        unsigned long long m32 = __builtin_amdgcn_ballot_w64(row_bytes <= half) & acts & ~m16;
        const unsigned long long cuts16 = __builtin_amdgcn_ballot_w64((jpos & 15u) == 0u) & acts;   // where pieces begin
        const unsigned long long cuts32 = __builtin_amdgcn_ballot_w64((jpos & 31u) == 0u) & acts;
        // Runs of many tokens go with the longer rows, whatever their length is: their search is made for all tokens at once there.
        // (many: where the next kManyTokens - 1 lanes continue the run.  Not in small batches: their 14 scalar instructions were 2 % of an
        // iteration at T = 15 M, K = 20,011, where a batch has 6 tokens)
        if (MODE == MODE_SAMPLE && n >= 2 * kManyTokens) {
            const unsigned long long more = ~starts & ~(~1ull << (n - 1));   // tokens that continue a run
            unsigned long long next = more >> 1;
            next &= next >> 1;
            next &= next >> 2;
            next &= next >> (kManyTokens - 5);
            const unsigned long long many = starts & next, inside = more | many;
            const unsigned long long lanes = (((inside + many) ^ inside) & inside) | many;   // (a carry runs from a start to the run's end)
            m16 &= ~lanes; m32 &= ~lanes;
        }
        // a pass serves four (two) runs at the cost of about one: a class that would not fill most of one pass goes
        // with the next wider one
        if (__builtin_popcountll(m16 & cuts16) < 3) { if (half >= quarter) m32 |= m16; m16 = 0ull; }
        if (__builtin_popcountll(m32 & cuts32) < 2) m32 = 0ull;
        const unsigned long long cm16 = m16 & cuts16, cm32 = m32 & cuts32;
        // longer rows: the tokens of those of one block (256 entries), and of several; the last token of each of their runs
        unsigned long long wide = __builtin_amdgcn_ballot_w64(row_bytes <= 16u * kWave) & acts & ~(m16 | m32);
        unsigned long long large = acts & ~(m16 | m32 | wide);
        const unsigned long long ends = alone ? acts : (starts >> 1) | (1ull << (n - 1));
        unsigned long long wide_ends = ends & wide, large_ends = ends & large;

        // ---- rows of at most 4 G entries: 64 / G runs at a time, one per group of G lanes ----
        // Token side: lane i holds token i of the batch.  Group side: the G lanes of group g hold the row of the
        // g-th run of the pass, 4 entries per lane.  Per class, the runs' row offsets and lengths are first packed
        // into the low lanes (slot r = r-th run of the class); a pass then pulls four (two) slots.
        auto run_class = [&](auto G_, const unsigned long long cm, const unsigned long long cuts, const bool in_class) {
            constexpr int G = decltype(G_)::value, NG = kWave / G, LG = G == 16 ? 4 : 5;
            const int nruns = (int)__builtin_popcountll(cm);   // wave-uniform
            if (nruns == 0) return;
            uint32_t zero = 0u;
            asm volatile("" : "+s"(zero));   // (keeps the compiler from running the set-up below ahead of this test)
            const int npass = (nruns + NG - 1) / NG;
            // (an opaque copy of the lane number: values derived from it are formed here, per class, instead of once
            // per kernel and then held in registers the kernel does not have to spare)
            uint32_t ln = (uint32_t)lane;
            asm volatile("" : "+v"(ln));
            const uint32_t gi = ln >> LG, li = ln & (uint32_t)(G - 1), li16 = li << 4;
            // Slot order: the pieces of one token first, the longer ones after them, each kind in batch order.  A pass
            // runs as many search steps as its longest piece has tokens, so like goes with like.  `rank` = 1 + slot of
            // the piece this lane belongs to.
            const unsigned long long sing = cm & ((cuts >> 1) | (1ull << (n - 1)));   // a piece that ends where the next begins
            const uint32_t nsing = (uint32_t)__builtin_popcountll(sing);
            const uint32_t rank = __builtin_amdgcn_inverse_ballot_w64(sing) ? bits_up_to_lane(sing)
                                                                            : nsing + bits_up_to_lane(cm & ~sing);
            // slots: a piece's first lane writes to slot rank - 1; all other lanes write to lane 63, which is a slot
            // only if every lane starts a piece
            const uint32_t dst4 = __builtin_amdgcn_inverse_ballot_w64(cm) ? (rank - 1u) << 2 : 252u + zero;
            const uint32_t slot_pk = lane_push(row_bytes | ((uint32_t)lane << 18), dst4);   // length | first token lane * 4 << 16
            const uint32_t slot_off = lane_push(row_off, dst4);
            const uint32_t my_piece = in_class ? rank - 1u : 0x80000000u;   // token side: piece of this token
            const uint32_t jg4 = (jpos & (uint32_t)(G - 1)) << 2;           // and its place in it, times 4
            constexpr unsigned long long ONES = G == 16 ? 0x0001000100010001ull : 0x0000000100000001ull;   // first lane of every group

            // Request the rows of the next pass.  Slots that no piece was put in read as rows of length 0, which move no data
            // (slot 63, and past the last of all, as some row of the batch): nothing is looked at of what a spare group gets.
            uint32_t slot4 = gi << 2;
            auto issue = [&](uint4 &blk, uint32_t &pk) {
                pk = lane_pull(slot_pk, slot4);
                const uint32_t off = lane_pull(slot_off, slot4);
                slot4 += (uint32_t)NG << 2;
                blk = load_rows_at(rows, li16 < (pk & 0xffffu) ? off + li16 : 0xffffffffu);
            };
            auto compute = [&](const int ps, const uint4 &cur, const uint32_t pk) {
                RowBlock b;
                block_products<STAGED, PACK, G>(cur, cbits, lds_phi, phi_row, b, ov);
                // S of the group's run in all its lanes
                const float S = G == 16 ? dpp_f32<0x15f, 0xf>(b.incl)                    // row_newbcast:15
                                        : half_last(b.incl);
                // token side: is this token's piece part of the pass, and which lane will hold its result
                const uint32_t gt = my_piece - (uint32_t)(ps * NG);
                const bool in_pass = gt < (uint32_t)NG;
                const uint32_t src4 = (gt << (LG + 2)) + jg4;
                uint32_t zacc = 0u;
                if (MODE == MODE_SAMPLE) {
                    const float base = b.incl - b.a3;
                    const float p0 = base + b.a0, p1 = base + b.a1, p2 = base + b.a2;
                    // the last lane of every group's row: if rounding leaves no lane, the choice falls on it (its padding
                    // repeats the row's last topic)
                    const unsigned long long sent = __builtin_amdgcn_ballot_w64(li16 + 16u == (pk & 0xffffu));
                    const unsigned long long pass_mask = __builtin_amdgcn_ballot_w64(in_pass);
                    // Lane j of a group collects the result of the j-th token of the group's piece.  `todo` marks the
                    // token lanes at position j of the pass's pieces: when it is empty, no piece is that long.
                    unsigned long long todo = pass_mask & cuts, collect = ONES;
                    uint32_t ua = pk >> 16;                           // lane * 4 of the token that is served next
                    uint32_t da = (uint32_t)(lane & ~(G - 1)) << 2;   // lane * 4 of the group lane that collects its result
                    float x = lane_pull(u1, ua) * S;
                    while (todo) {
                        // problem 1 for one token per group: position of x in the prefix sums of P.  (Whether the
                        // token takes this branch is decided on the token side, once S has arrived there.)
                        ua += 4u;
                        const float x_next = lane_pull(u1, ua) * S;
                        const unsigned long long ge = __builtin_amdgcn_ballot_w64(b.incl >= x) | sent;
                        const unsigned long long win = ge & ~(ge - ONES);   // first such lane of every group
                        uint32_t sel = cur.w;
                        sel = p2 >= x ? cur.z : sel;
                        sel = p1 >= x ? cur.y : sel;
                        sel = p0 >= x ? cur.x : sel;
                        // the winning lane writes to the collecting lane, every other lane to the collecting lane's
                        // neighbour, whose own turn to collect is another one
                        const uint32_t got = lane_push(sel, da + (__builtin_amdgcn_inverse_ballot_w64(win) ? 0u : 4u));
                        zacc = __builtin_amdgcn_inverse_ballot_w64(collect) ? got : zacc;
                        da += 4u; collect <<= 1;
                        todo = (todo << 1) & pass_mask & ~cuts;
                        x = x_next;
                    }
                }
                const float St = lane_pull(S, src4);
                my_S = in_pass ? St : my_S;
                if (MODE == MODE_SAMPLE) {
                    const uint32_t zt = lane_pull(zacc, src4);
                    my_z = in_pass ? zt : my_z;
                }
            };
            uint4 blk_a, blk_b; uint32_t pk_a, pk_b;
            issue(blk_a, pk_a);
            for (int ps = 0;; ps += 2) {
                issue(blk_b, pk_b);
                compute(ps, blk_a, pk_a);
                if (ps + 1 >= npass) break;
                issue(blk_a, pk_a);
                compute(ps + 1, blk_b, pk_b);
                if (ps + 2 >= npass) break;
            }
        };
        // The same by way of the wavefront's part of LDS.  Bound by LDS: a lane permutation takes 6.1 cycles of it, a read of a few
        // places 2.3 and a write by a few lanes 4.1: 42 cycles instead of 79 for two rows of at most 128 entries.
        const uint32_t tok_at = SLOTS ? (uint32_t)(((q->K + 3) & ~3) + 4 + ((q->n3 + 3) & ~3)) * 4u + (uint32_t)wave * kSlotBytes : 0u;
        typedef uint32_t pair_t __attribute__((ext_vector_type(2)));
        typedef __attribute__((address_space(3))) pair_t lds_pair;
        typedef __attribute__((address_space(3))) uint32_t lds_word;
        auto run_class_slots = [&](auto G_, const unsigned long long in_class, const unsigned long long cm, const unsigned long long cuts) {
            constexpr int G = decltype(G_)::value, NG = kWave / G, LG = G == 16 ? 4 : 5;
            const int nruns = (int)__builtin_popcountll(cm);   // wave-uniform
            if (nruns == 0) return;
            const int npass = (nruns + NG - 1) / NG;
            uint32_t ln = (uint32_t)lane;
            asm volatile("" : "+v"(ln));
            // Slot order as above.  The last token of every piece puts down its slot: the row's length, the piece's tokens, its
            // first token; the row's offset.
            const unsigned long long lasts = ((cuts >> 1) | (1ull << (n - 1))) & in_class, sing = cm & lasts;
            const uint32_t rank1 = bits_up_to_lane(sing), rank2 = (uint32_t)__builtin_popcountll(sing) + bits_up_to_lane(cm & ~sing);
            const uint32_t piece_at = tok_at + kWave * 4u - 8u;
            const uint32_t mine_at = piece_at + (__builtin_amdgcn_inverse_ballot_w64(sing) ? rank1 : rank2) * 8u;
            const uint32_t jp = jpos & (uint32_t)(G - 1);
            if (__builtin_amdgcn_inverse_ballot_w64(lasts))
                *(lds_pair *)mine_at = pair_t{row_bytes | ((jp + 1u) << 16) | ((ln - jp) << 26), row_off};
            if (__builtin_amdgcn_inverse_ballot_w64((1ull << (2 * NG)) - 1ull))   // spare ones: rows of length 0
                *(lds_pair *)(piece_at + (uint32_t)(nruns + 1) * 8u + ln * 8u) = pair_t{0u, 0u};
            wave_lds_fence();
            constexpr unsigned long long ONES = G == 16 ? 0x0001000100010001ull : 0x0000000100000001ull;   // first lane of every group
            const uint32_t li16 = (ln & (uint32_t)(G - 1)) << 4;
            uint32_t slot_at = piece_at + 8u + (ln >> LG) * 8u;   // of the pass that is computed
            auto issue = [&](const int ahead, uint4 &blk, uint32_t &pk) {
                const pair_t w = *(lds_pair *)(slot_at + (uint32_t)(ahead * NG) * 8u);
                pk = w.x;
                blk = load_rows_at(rows, li16 < (w.x & 0xffffu) ? w.y + li16 : 0xffffffffu);
            };
            auto compute = [&](const uint4 &cur, const uint32_t pk) {
                uint32_t at = tok_at + (pk >> 24);               // place of the token that is served next
                float u = __uint_as_float(*(lds_word *)at);
                RowBlock b;
                block_products<STAGED, PACK, G>(cur, cbits, lds_phi, phi_row, b, ov);
                const float S = G == 16 ? dpp_f32<0x15f, 0xf>(b.incl) : half_last(b.incl);
                if (__builtin_amdgcn_inverse_ballot_w64(ONES << (G - 1))) *(lds_word *)slot_at = __float_as_uint(b.incl);
                slot_at += (uint32_t)NG * 8u;
                const float base = b.incl - b.a3;
                const float p0 = base + b.a0, p1 = base + b.a1, p2 = base + b.a2;
                // the last lane of every group's row: if rounding leaves no lane, the choice falls on it
                const unsigned long long sent = __builtin_amdgcn_ballot_w64(li16 + 16u == (pk & 0xffffu));
                unsigned long long act = __builtin_amdgcn_ballot_w64(((pk >> 16) & 0xffu) > 0u);   // groups whose piece has a token left
                for (uint32_t j = 1;; j++) {
                    const float x = u * S;
                    const unsigned long long ge = __builtin_amdgcn_ballot_w64(b.incl >= x) | sent;
                    const unsigned long long win = ge & ~(ge - ONES) & act;   // first such lane of every group
                    uint32_t sel = cur.w;
                    sel = p2 >= x ? cur.z : sel;
                    sel = p1 >= x ? cur.y : sel;
                    sel = p0 >= x ? cur.x : sel;
                    if (__builtin_amdgcn_inverse_ballot_w64(win)) *(lds_word *)at = sel;
                    act = __builtin_amdgcn_ballot_w64(((pk >> 16) & 0xffu) > j);
                    if (!act) break;
                    at += 4u;
                    u = __uint_as_float(*(lds_word *)at);
                }
            };
            uint4 blk_a, blk_b; uint32_t pk_a, pk_b;
            issue(0, blk_a, pk_a);
            for (int ps = 0;; ps += 2) {
                issue(1, blk_b, pk_b);
                compute(blk_a, pk_a);
                if (ps + 1 >= npass) break;
                issue(1, blk_a, pk_a);
                compute(blk_b, pk_b);
                if (ps + 2 >= npass) break;
            }
            wave_lds_fence();
            const float St = __uint_as_float(*(lds_word *)mine_at);
            my_S = __builtin_amdgcn_inverse_ballot_w64(in_class) ? St : my_S;
        };
        // ---- longer rows: one run at a time over the whole wavefront ----
        // `cur` holds the run's row (its first block), `last` the number of the row's last piece of 16 bytes; the next run's row
        // is fetched into `nxt` before this run's arithmetic starts.  Rows of several blocks have a loop of their own, so that
        // no load that is made for a longer row only is waited for on the way of the others.
        float Qv = Q;
        asm volatile("" : "+v"(Qv));   // (beside a run's S, which is in a scalar register, an addition takes no second one)
        int lane16 = lane * 16;
        // The row is a piece of the chunk's rows: its offset is the load's scalar one, its end the descriptor's length, so a lane
        // past the end reads zeros and moves no data.
        auto row_at = [&](const int last, const uint32_t off) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(rows_base), (short)0, (int)(off + (uint32_t)(last + 1) * 16u), 0x00020000);
        };
        auto fetch = [&](const int e, uint4 &blk, int &last, uint32_t &off) {
            // Requested without any branch around the load: a load inside a branch would make the compiler wait for ALL
            // outstanding loads where the branches meet, i.e. for the row just requested, before the current run's
            // arithmetic.  Without a further run (e < 0) it is lane 63's row, which the batch has read as a rule, or nothing.
            // (Batches of the other modes may have a token or two of 64, and then it is nothing: see below.)
            last = (int)readlane_u32((uint32_t)row_last, e);
            if (MODE != MODE_SAMPLE) last = e < 0 ? -1 : last;
            off = readlane_u32(row_off, e);
            asm volatile("" : "+v"(lane16));
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(row_at(last, off), lane16, (int)off, 0);
            blk = make_uint4(v[0], v[1], v[2], v[3]);
        };
        // block 1, 2, ... of the same row (past its end: zeros, and no data moves)
        auto fetch_more = [&](const int last, const uint32_t off, const int block) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(row_at(last, off), lane16, (int)(off + (uint32_t)block * 16u * kWave), 0);
            return make_uint4(v[0], v[1], v[2], v[3]);
        };
        // the first rows are requested now, so that they arrive while the short rows are worked on
        int e_a = first_bit(wide_ends), e_b, e_c = first_bit(large_ends), e_d, last_a, last_b, last_c, last_d;
        uint32_t off_a, off_b, off_c, off_d;
        uint4 blk_a, blk_b, blk_c, blk_c2, blk_d, blk_d2;
        fetch(e_a, blk_a, last_a, off_a);
        // (Not those of several blocks where nothing is sampled: few batches have any, and with marks the loads are most of what a batch
        // costs.  S and Q of 3,000 tokens of T = 10 M, K = 12,000 182 -> 177 us, of 200,000 547 -> 542.)
        if (MODE == MODE_SAMPLE) {
            fetch(e_c, blk_c, last_c, off_c);
            blk_c2 = fetch_more(last_c, off_c, 1);
        }

        if (SLOTS) {
            if (m16 | m32) {
                lds_word *mine = (lds_word *)(tok_at + (uint32_t)lane * 4u);
                *mine = __float_as_uint(u1);
                wave_lds_fence();
                run_class_slots(std::integral_constant<int, 16>{}, m16, cm16, cuts16);
                run_class_slots(std::integral_constant<int, 32>{}, m32, cm32, cuts32);
                wave_lds_fence();
                my_z = *mine;
            }
        } else {
            run_class(std::integral_constant<int, 16>{}, cm16, cuts16, __builtin_amdgcn_inverse_ballot_w64(m16));
            run_class(std::integral_constant<int, 32>{}, cm32, cuts32, __builtin_amdgcn_inverse_ballot_w64(m32));
        }
        if (MODE == MODE_SAMPLE && (m16 | m32)) {
            // the coin of the tokens served above, all at once
            sparse_mask = __builtin_amdgcn_ballot_w64(u0 * (my_S + Q) < my_S) & (m16 | m32);
        }

        // ---- longer rows (the first fetches went out above) ----
        // Bound by instructions of both kinds: the vector unit takes 2.5 cycles (additions, shifts, products) or 4.3 to 4.6 (compares,
        // DPP, SDWA, conversions, lane moves), and the scalar unit, one for a CU's four SIMDs, 4.3 per SIMD.  So the masks are walked
        // by the runs' last tokens (a dozen scalar instructions per run and six per token, where a walk by first tokens took
        // 42 and 8), and rows of one block share no code with longer ones.  Sampling pass, late iterations, with the shift in phi_of: T = 10 M,
        // K = 1,000 0.61 -> 0.56 ms, T = 100 M, K = 10,000 6.71 -> 6.43.
        // Takes the run that ends at lane e out of `tokens`: the lanes of the run (those before it have been taken).
        auto take_run = [&](const int e, unsigned long long &tokens) {
            const unsigned long long beyond = ~1ull << e, run = tokens & ~beyond;
            tokens &= beyond;
            return run;
        };
        auto do_wide = [&](const int e, const uint4 &cur, const int last, int &e_next, uint4 &nxt, int &nxt_last, uint32_t &nxt_off) {
            wide_ends = clear_bit(wide_ends, e);
            e_next = first_bit(wide_ends);
            fetch(e_next, nxt, nxt_last, nxt_off);
            __builtin_amdgcn_sched_barrier(0);      // (left to the compiler the request goes out after the wait for this run's row:
                                                    // log-likelihood at T = 10 M, K = 12,000 500 -> 472 us, sampling 0 to 0.7 %)
            const unsigned long long in_run = take_run(e, wide);
            // element-wise product A_d (.) Bhat_v, its prefix sums and its sum S (Alg. 2, product loop)
            RowBlock b;
            block_products<STAGED, PACK>(cur, cbits, lds_phi, phi_row, b, ov);
            const float S = readlane_f32(b.incl, 63);
            if (MODE != MODE_SAMPLE) {
                if (__builtin_amdgcn_inverse_ballot_w64(in_run)) my_S = S;
                return;
            }
            // every lane evaluates the coin and the position for its own token; lanes of this run are used
            unsigned long long sparse = __builtin_amdgcn_ballot_w64(u0 * (S + Qv) < S) & in_run;
            sparse_mask |= sparse;                  // problem 2 is served after the runs, four tokens at a time
            if (sparse) {
                const float xs = u1 * S;
                const float base = b.incl - b.a3;
                const float p0 = base + b.a0, p1 = base + b.a1, p2 = base + b.a2;
                if ((int)__builtin_popcountll(sparse) >= kManyTokens) {
                    // many tokens: every lane looks for its own.  "First lane whose sum reaches x" is the same over the sums' running
                    // maximum, which rounding leaves in order, and a search by halves of that finds it.
                    const int top = wave_incl_scan_max(__float_as_int(b.incl));
                    // 4 times the lane; the first step tells the halves apart (half of 128 is a constant an instruction can hold)
                    uint32_t at4 = readlane_f32(__int_as_float(top), 31) < xs ? 64u : 0u;
                    asm volatile("" : "+v"(at4));
                    at4 <<= 1;
#pragma unroll
                    for (uint32_t half = 16u; half; half >>= 1)
                        at4 = __int_as_float((int)lane_pull((uint32_t)top, at4 + (half - 1u) * 4u)) < xs ? at4 + half * 4u : at4;
                    at4 = min(at4, (uint32_t)last * 4u);
                    uint32_t sel = lane_pull(cur.w, at4);
                    const uint32_t s2 = lane_pull(cur.z, at4), s1 = lane_pull(cur.y, at4), s0 = lane_pull(cur.x, at4);
                    sel = lane_pull(p2, at4) >= xs ? s2 : sel;
                    sel = lane_pull(p1, at4) >= xs ? s1 : sel;
                    sel = lane_pull(p0, at4) >= xs ? s0 : sel;
                    my_z = __builtin_amdgcn_inverse_ballot_w64(sparse) ? sel : my_z;
                } else do {
                    // problem 1: position of x in the prefix sums of P.  If rounding leaves no lane of the row's, the choice falls
                    // on its last one, whose padding repeats the row's last topic
                    const int r = first_bit(sparse);
                    sparse = clear_bit(sparse, r);
                    const float x = readlane_f32(xs, r);
                    const int L = (int)min((uint32_t)first_bit(__builtin_amdgcn_ballot_w64(b.incl >= x)), (uint32_t)last);
                    uint32_t sel = cur.w;
                    sel = p2 >= x ? cur.z : sel;
                    sel = p1 >= x ? cur.y : sel;
                    sel = p0 >= x ? cur.x : sel;
                    my_z = llvm_amdgcn_writelane_u32(readlane_u32(sel, L), (unsigned)r, my_z);
                } while (sparse);
            }
        };
        auto do_large = [&](const int e, const uint4 &cur, const uint4 &cur2, const int last, const uint32_t off, int &e_next, uint4 &nxt,
                            uint4 &nxt2, int &nxt_last, uint32_t &nxt_off) {
            large_ends = clear_bit(large_ends, e);
            e_next = first_bit(large_ends);
            fetch(e_next, nxt, nxt_last, nxt_off);
            nxt2 = fetch_more(nxt_last, nxt_off, 1);
            __builtin_amdgcn_sched_barrier(0);
            const unsigned long long in_run = take_run(e, large);
            RowBlock b0, b1;
            block_products<STAGED, PACK>(cur, cbits, lds_phi, phi_row, b0, ov);
            block_products<STAGED, PACK>(cur2, cbits, lds_phi, phi_row, b1, ov);
            const float t0 = readlane_f32(b0.incl, 63);
            float S = t0 + readlane_f32(b1.incl, 63);
            float through = S;      // lane i: sum through block i, from the second on (rows of up to 64 blocks)
            const int nblk = (last >> 6) + 1;
            if (nblk > 2) {
                // The row of a long document, in the first iterations above all: one block after the other, the next one
                // requested before the arithmetic of this.  The sums through each are kept, so that a draw reads only the
                // block that holds it.  First iteration at T = 15 M, K = 20,011 (documents of 1,000 tokens, weighted by
                // length): 7.0 -> 5.1 ms, at T = 100 M, K = 10,000 20.0 -> 19.0.  (Requested before the second block's
                // arithmetic, and then by rows of two blocks too, the third one costs later iterations 1 %.)
                through = __builtin_amdgcn_inverse_ballot_w64(2ull) ? S : -1.f;
                uint4 en = fetch_more(last, off, 2);
                for (int blk = 2; blk < nblk; blk++) {
                    const uint4 ec = en;
                    if (blk + 1 < nblk) en = fetch_more(last, off, blk + 1);
                    RowBlock bb;
                    block_products<STAGED, PACK>(ec, cbits, lds_phi, phi_row, bb, ov);
                    S = S + readlane_f32(bb.incl, 63);
                    if (MODE == MODE_SAMPLE && blk < kWave)
                        through = __uint_as_float(llvm_amdgcn_writelane_u32(__float_as_uint(S), (unsigned)blk, __float_as_uint(through)));
                }
            }
            if (MODE != MODE_SAMPLE) {
                if (__builtin_amdgcn_inverse_ballot_w64(in_run)) my_S = S;
                return;
            }
            unsigned long long sparse = __builtin_amdgcn_ballot_w64(u0 * (S + Qv) < S) & in_run;
            sparse_mask |= sparse;
            const float xs = u1 * S;
            while (sparse) {
                const int r = first_bit(sparse);
                sparse = clear_bit(sparse, r);
                const float x = readlane_f32(xs, r);
                uint32_t sel;
                if (t0 >= x) sel = search_block(cur, b0, 0.f, x, kWave * 4);
                else if (nblk == 2 || readlane_f32(through, 1) >= x) sel = search_block(cur2, b1, t0, x, 4 * (last + 1 - kWave));
                else {
                    // the block that holds the position is known from the sums above (beyond 64 blocks it is looked for)
                    const unsigned long long reach = __builtin_amdgcn_ballot_w64(through >= x);
                    int blk = reach ? (int)__builtin_ctzll(reach) : min(nblk, kWave) - 1;
                    float carry = readlane_f32(through, blk - 1);
                    sel = 0u;
                    for (; blk < nblk; blk++) {
                        const uint4 ec = fetch_more(last, off, blk);
                        RowBlock bb;
                        block_products<STAGED, PACK>(ec, cbits, lds_phi, phi_row, bb, ov);
                        const float tot = readlane_f32(bb.incl, 63);
                        if (blk == nblk - 1 || carry + tot >= x) { sel = search_block(ec, bb, carry, x, 4 * (last + 1 - blk * kWave)); break; }
                        carry = carry + tot;
                    }
                }
                my_z = llvm_amdgcn_writelane_u32(sel, (unsigned)r, my_z);
            }
        };

        if (wide) {
            for (;;) {
                do_wide(e_a, blk_a, last_a, e_b, blk_b, last_b, off_b);
                if (!wide_ends) break;
                do_wide(e_b, blk_b, last_b, e_a, blk_a, last_a, off_a);
                if (!wide_ends) break;
            }
        }
        if (large) {
            if (MODE != MODE_SAMPLE) {
                fetch(e_c, blk_c, last_c, off_c);
                blk_c2 = fetch_more(last_c, off_c, 1);
            }
            for (;;) {
                do_large(e_c, blk_c, blk_c2, last_c, off_c, e_d, blk_d, blk_d2, last_d, off_d);
                if (!large_ends) break;
                do_large(e_d, blk_d, blk_d2, last_d, off_d, e_c, blk_c, blk_c2, last_c, off_c);
                if (!large_ends) break;
            }
        }
        unsigned long long dense_mask = 0ull;
        if (MODE == MODE_SAMPLE) {
            my_z >>= cbits;                               // (so far the entries that the draws fell on)
            dense_mask = acts & ~sparse_mask;
        }

        // The token's number is read again rather than carried through the batch in a register (the kernel is at its
        // register limit; the 4 bytes come from a cache line this wavefront loaded at the top of the batch).  Requested
        // here, it arrives while the dense branch below is served.
        uint32_t t_late = 0u;
        q = params_again();
        auto *tile_now = const_mem(q->tiles + tile_at);
        if (MODE != MODE_LOGLIK) {
            uint32_t pos_t = (uint32_t)(batch + lane);
            asm volatile("" : "+v"(pos_t));
            if (act) t_late = q->tok_t[tile_now->begin + (int)pos_t];
        }

        if (MODE == MODE_SAMPLE && dense_mask) {
            // problem 2 for the tokens whose coin chose it: DPP row g (16 lanes) serves the g-th of up to four tokens
            const int K = q->K, n3 = q->n3, K4 = (K + 3) & ~3;
            const double *l3_64_row = q->l3_64 + (size_t)tile_now->word * (size_t)n3;
            if (lane == 0) atomicAdd(reinterpret_cast<unsigned int *>(lds_phi + (STAGED ? K4 : 0)) + 1, (unsigned int)__builtin_popcountll(dense_mask));   // statistic only
            if (q->alias_table != nullptr) {   // (every word then keeps a dense row)
                // Walker's alias method for all these tokens at once: the bucket is floor(u1 K), taken in integers from
                // the 24 random bits behind u1; the bucket's own topic if the fraction of u1 K lies below its
                // probability, its alias otherwise
                const uint32_t bits24 = (uint32_t)(u1 * 16777216.0f);
                const uint32_t lo = bits24 * (uint32_t)K, hi = __umulhi(bits24, (uint32_t)K);
                const uint32_t bucket = (hi << 8) | (lo >> 24);
                const float frac = (float)(lo & 0xffffffu) * (1.0f / 16777216.0f);
                if (__builtin_amdgcn_inverse_ballot_w64(dense_mask)) {
                    const uint2 e = q->alias_table[(size_t)tile_now->row * (size_t)K + bucket];
                    my_z = frac < __uint_as_float(e.x) ? bucket : e.y;
                }
                dense_mask = 0ull;
            }
            const float xd = u1 * sum_w;
            uint32_t ln = (uint32_t)lane;
            asm volatile("" : "+v"(ln));               // (as above: lane-derived values formed where they are used)
            const uint32_t g = ln >> 4, li = ln & 15u;
            if (STAGED) {
                int l3_top_shift = 0;   // the descent over l3 starts with stride 16^(l3_top_shift / 4)
                while ((16 << l3_top_shift) < n3) l3_top_shift += 4;
                while (dense_mask) {
                    // the next four tokens (fewer at the end: the spare rows then repeat the first token's query, and
                    // arrive at the same answer)
                    const unsigned long long before = dense_mask;
                    uint32_t tl[4];
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        tl[q] = dense_mask ? (uint32_t)__builtin_ctzll(dense_mask) : tl[0];
                        if (dense_mask) dense_mask = clear_bit(dense_mask, (int)tl[q]);
                    }
                    // lane number * 4 of the row's token: the four of them packed into one scalar, a byte each
                    const uint32_t packed = (tl[0] | (tl[1] << 8) | (tl[2] << 16) | (tl[3] << 24)) << 2;
                    const uint32_t mine4 = __builtin_amdgcn_ubfe(packed, g << 3, 8u);
                    const float x = lane_pull(xd, mine4);
                    const uint32_t k = dense_query4_staged((uint32_t)K4 * 4u, (uint32_t)K4 * 4u + 16u, l3_64_row, n3, l3_top_shift, K,
                                                           x, li, ln & 48u);
                    // all 16 lanes of a row hold the row's answer and send it to the row's token
                    const uint32_t got = lane_push(k, mine4);
                    my_z = __builtin_amdgcn_inverse_ballot_w64(before ^ dense_mask) ? got : my_z;
                }
            }
            while (dense_mask) {
                int tl[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    tl[q] = dense_mask ? (int)__builtin_ctzll(dense_mask) : -1;
                    if (dense_mask) dense_mask = clear_bit(dense_mask, tl[q]);
                }
                const int mine = g == 0 ? tl[0] : g == 1 ? tl[1] : g == 2 ? tl[2] : tl[3];
                const float x = __int_as_float(__builtin_amdgcn_ds_bpermute((mine < 0 ? lane : mine) << 2, __float_as_int(xd)));
                const uint32_t k = dense_query4(phi_row, q->Kpad, q->l3 + (size_t)tile_now->word * (size_t)q->n3pad, l3_64_row, n3, K, x, (int)li, ov);
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if (tl[q] >= 0) my_z = llvm_amdgcn_writelane_u32(readlane_u32(k, 16 * q), (unsigned)tl[q], my_z);
            }
        }

        if (act) {
            if (MODE == MODE_SAMPLE) {
                reinterpret_cast<ZT *>(q->z)[q->z_rel + (int64_t)t_late] = (ZT)my_z;
                // the second copy, in word-major order, is what CountByVZ reads (coalesced here and there)
                uint32_t pos = (uint32_t)(batch + lane);   // of the token inside the tile
                asm volatile("" : "+v"(pos));
                reinterpret_cast<ZT *>(q->z_wm)[tile_now->wm_begin + (int64_t)pos] = (ZT)my_z;
            } else if (MODE == MODE_PROBS) {
                const uint32_t at = q->marks ? token_number(q->marks[t_late >> 5], t_late) : t_late;
                q->out_S[at] = my_S; q->out_Q[at] = Q;
            } else {
                ll_acc += log((double)(my_S + Q));
            }
        }
        // the next batch: taken from the ticket counter, as wavefronts become free.  (Asking for it and for its tokens'
        // records earlier, before the dense branch, changed nothing.)
        int ticket = 0;
        if (MODE == MODE_LOGLIK) ticket = (round + 1) * nwaves + wave;   // fixed assignment: the sums come out bit-identical every time
        else if (lane == 0) ticket = atomicAdd(reinterpret_cast<int *>(lds_phi + (STAGED ? (q->K + 3) & ~3 : 0)), 1);   // (handed out as wavefronts become free)
        batch = __builtin_amdgcn_readfirstlane(ticket) * bs;   // wave-uniform: loop control stays scalar
        if (batch >= count) break;
        q = params_again();
        d = -1; t = 0u; rec = make_uint2(q->row_unit0, 0u);
        if (lane < min(bs, count - batch)) {
            const int at = tile_now->begin + batch + lane;
            d = q->tok_doc[at];
            t = q->tok_t[at];
            rec = q->docrec[d];
        }
    }

    if (MODE == MODE_LOGLIK) {
        double tot = readlane_f64(wave_incl_scan(ll_acc), 63);
        if (lane == 0) ll_wave[wave] = tot;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int w = 0; w < nwaves; w++) sum += ll_wave[w];
            p.out_ll[tile_at] = sum;
        }
    }
    if (!kWalks || !light) break;
    EStepParamsConst *q = params_again();
    const int next_at = tile_at + q->walkers;
    if (next_at >= q->n_tiles) break;
    // The next light word.  Everything its start needs from memory is requested before the barrier at which the workgroup's
    // wavefronts come together; then the last word's topics get their base values back - the whole row is staged again where they
    // are more than one per thread - and the new word's take their place.
    auto *rec0 = const_mem(q->wrec + const_mem(q->tiles + tile_at)->row);
    tile_at = next_at;
    auto *tile = const_mem(q->tiles + tile_at);
    auto *rec1 = const_mem(q->wrec + tile->row);
    const uint2 wr0 = make_uint2(rec0->x, rec0->y), wr = make_uint2(rec1->x, rec1->y);
    const uint32_t *ent0 = q->lw_ent + (size_t)wr0.x * 32u, *ent = q->lw_ent + (size_t)wr.x * 32u;
    const float *val = q->lw_phi + (size_t)wr.x * 32u;
    const float *l3_row = q->l3 + (size_t)tile->word * (size_t)q->n3pad;
    count = tile->count;
    bs = (count + nwaves - 1) / nwaves;
    bs = __builtin_amdgcn_readfirstlane(bs > kWave ? kWave : bs);
    batch = wave * bs;
    d = -1; t = 0u; rec = make_uint2(q->row_unit0, 0u);
    if (lane < min(bs, count - batch)) {
        d = q->tok_doc[tile->begin + batch + lane];
        t = q->tok_t[tile->begin + batch + lane];
    }
    const int tid = wave * kWave + lane;
    const int nt = (int)blockDim.x, n3 = q->n3, K4 = (q->K + 3) & ~3;
    float *lds_l3 = lds_phi + K4 + 4;
    const bool restore = (int)wr0.y <= nt;
    uint32_t k0 = 0u, e = 0u;
    float b0 = 0.f, v = 0.f, c = 0.f;
    if (tid < (int)wr.y) { e = ent[tid]; v = val[tid]; }
    if (restore && tid < (int)wr0.y) { k0 = ent0[tid] >> cbits; b0 = q->base[k0]; }
    if (tid < n3) c = l3_row[tid];
    if (d >= 0) rec = q->docrec[d];
    sum_w = *const_mem(q->sumphi + tile->word);
    Q = first_lane(q->alpha * sum_w);
    lds_barrier();
    if (restore) { if (tid < (int)wr0.y) lds_phi[k0] = b0; }
    else {   // (two loads at a time: d, t and rec are in registers)
        const float4 *src = reinterpret_cast<const float4 *>(q->base);
        float4 *dst = reinterpret_cast<float4 *>(lds_phi);
        const int nq = K4 / 4;
        for (int i = tid; i < nq; i += 2 * nt) {
            const float4 f0 = src[i], f1 = src[min(i + nt, nq - 1)];
            dst[i] = f0; dst[min(i + nt, nq - 1)] = f1;
        }
    }
    if (tid < n3) lds_l3[tid] = c;
    for (int i = tid + nt; i < n3; i += nt) lds_l3[i] = l3_row[i];
    int first_ticket = nwaves;
    asm volatile("" : "+s"(first_ticket));   // (not held in a vector register over the tiles)
    if (tid == 0) reinterpret_cast<int *>(lds_phi)[K4] = first_ticket;
    lds_barrier();
    if (tid < (int)wr.y) lds_phi[e >> cbits] = v;
    for (int j = tid + nt; j < (int)wr.y; j += nt) lds_phi[ent[j] >> cbits] = val[j];
    lds_barrier();
    }

    if (MODE == MODE_SAMPLE) {
        __syncthreads();
        EStepParamsConst *q = params_again();
        const unsigned int wg_dense = reinterpret_cast<unsigned int *>(lds_phi + (STAGED ? (q->K + 3) & ~3 : 0))[1];   // dense-branch tokens of this workgroup
        if (threadIdx.x == 0 && wg_dense) atomicAdd(q->n_dense + (blockIdx.x & (kDenseSlots - 1)), (unsigned long long)wg_dense);
    }
}

// The bottom tree level (inclusive binary32 prefix sums of one Bhat row), rebuilt as the sampler's dense branch
// sees it; one wavefront per (row, 64-topic block).  rows[m][K] holds the Bhat rows of words[m].  Export / test aid.
__global__ void prefix_export_kernel(const float *rows, const double *l3_64, const int32_t *words, int m, int K, int n3,
                                     float *out) {
    const int nblk = (K + kWave - 1) / kWave;
    const int item = blockIdx.x, wi = item / nblk, blk = item % nblk, lane = lane_id();
    if (wi >= m) return;
    const size_t v = (size_t)words[wi];
    const int k = blk * kWave + lane;
    const double base = blk > 0 ? l3_64[v * (size_t)n3 + (size_t)(blk - 1)] : 0.0;
    const float f = k < K ? rows[(size_t)wi * (size_t)K + (size_t)k] : 0.f;
    const float c = (float)(base + wave_incl_scan((double)f));
    if (k < K) out[(size_t)wi * (size_t)K + (size_t)k] = c;
}

// ---------------------------------------------------------------------------------------------
// Histograms of the assignments by slabs: the topic totals C_k = sum_v B_vk, computed as the histogram of z (same numbers,
// 20x fewer bytes than column sums of B at K = 10^4), and CountByVZ for the long dense rows of B.  The assignments
// arrive word-major (z_wm), so a word's tokens are one contiguous segment; it is cut into slabs and each workgroup
// histograms one slab in LDS and adds the non-zero bins to the word's row: at most min(slab, K) global atomics per slab
// instead of one per token.  The first n_tot workgroups of a grid row take the totals' shares of z, the others the
// slabs; grid row y counts the topics [y range, (y + 1) range).  Totals and rows must be zero on entry
// (denominators_kernel and the Bhat kernel clear them after reading).
// ---------------------------------------------------------------------------------------------
struct VzItem { int32_t row; int32_t count; int64_t begin; };   // slab: count tokens from z_wm[begin] on

// f(topic) for each of the n assignments at zs, nt threads sharing the work (this is thread i0): 16-byte loads (8 or 4
// assignments per lane and load) over the aligned middle, single loads for the unaligned head and the tail.
// A one-assignment-per-load loop is bound by the latency of its dependent loads, not by bandwidth.
template <typename ZT, typename F>
__device__ __forceinline__ void for_each_z(const ZT *__restrict__ zs, int64_t n, int i0, int nt, F f) {
    constexpr int kPer = 16 / (int)sizeof(ZT);
    int64_t head = (int64_t)(((16u - (unsigned)(reinterpret_cast<uintptr_t>(zs) & 15u)) & 15u) / sizeof(ZT));
    if (head > n) head = n;
    for (int64_t i = i0; i < head; i += nt) f((uint32_t)zs[i]);
    const int64_t nvec = (n - head) / kPer;
    const uint4 *__restrict__ v = reinterpret_cast<const uint4 *>(zs + head);
    // the next 16 bytes are requested before the current ones are handed to f: f's work (LDS atomics, as a rule)
    // does not depend on them, so their latency passes under it
    int64_t j = i0;
    uint4 q = make_uint4(0u, 0u, 0u, 0u);
    if (j < nvec) q = v[j];
    while (j < nvec) {
        const int64_t jn = j + nt;
        uint4 qn = make_uint4(0u, 0u, 0u, 0u);
        if (jn < nvec) qn = v[jn];
        if (sizeof(ZT) == 2) {
            f(q.x & 0xffffu); f(q.x >> 16); f(q.y & 0xffffu); f(q.y >> 16);
            f(q.z & 0xffffu); f(q.z >> 16); f(q.w & 0xffffu); f(q.w >> 16);
        } else {
            f(q.x); f(q.y); f(q.z); f(q.w);
        }
        q = qn; j = jn;
    }
    for (int64_t i = head + nvec * kPer + i0; i < n; i += nt) f((uint32_t)zs[i]);
}

template <typename ZT, typename F>
__device__ __forceinline__ void block_for_each_z(const ZT *__restrict__ zs, int64_t n, F f) { for_each_z(zs, n, (int)threadIdx.x, (int)blockDim.x, f); }

// hist[k - k0] = assignments of topic k in [k0, k0 + n) among the len at zs; add(k - k0, count) for those that are not zero.
template <typename ZT, typename F>
__device__ __forceinline__ void count_slab(const ZT *__restrict__ zs, int64_t len, uint32_t *hist, int k0, int n, bool all_topics, F add) {
    for (int k = threadIdx.x; k < n; k += blockDim.x) hist[k] = 0u;
    __syncthreads();
    if (all_topics) block_for_each_z(zs, len, [&](uint32_t k) { atomicAdd(&hist[k], 1u); });
    else block_for_each_z(zs, len, [&](uint32_t k) { if (k - (uint32_t)k0 < (uint32_t)n) atomicAdd(&hist[k - (uint32_t)k0], 1u); });
    __syncthreads();
    for (int k = threadIdx.x; k < n; k += blockDim.x)
        if (const uint32_t h = hist[k]) add(k, h);
}

template <typename ZT>
__global__ void __launch_bounds__(1024) count_slabs_kernel(const ZT *z, int64_t T, int64_t per_block, int n_tot, unsigned long long *tot,
                                                           const VzItem *items, const ZT *z_wm, int32_t *cwk, int K, int Kpad, int range) {
    extern __shared__ uint32_t slab_hist[];
    const int k0 = (int)blockIdx.y * range, n = min(range, K - k0);
    if ((int)blockIdx.x < n_tot) {
        const int64_t first = (int64_t)blockIdx.x * per_block;
        count_slab(z + first, min(per_block, T - first), slab_hist, k0, n, gridDim.y == 1, [&](int k, uint32_t h) { atomicAdd(&tot[k0 + k], (unsigned long long)h); });
    } else {
        const VzItem it = items[(int)blockIdx.x - n_tot];
        int32_t *row = cwk + (size_t)it.row * (size_t)Kpad + k0;
        count_slab(z_wm + it.begin, (int64_t)it.count, slab_hist, k0, n, gridDim.y == 1, [&](int k, uint32_t h) { atomicAdd(&row[k], (int)h); });
    }
}

// Host streaming: a chunk's assignments in document order (relative to the chunk's first token) out of the
// word-major copy; the inverse of fill_zwm_kernel.
template <typename ZT>
__global__ void scatter_zwm_kernel(const Tile *tiles, const uint32_t *tok_t, const ZT *z_wm, ZT *z_chunk) {
    const Tile tile = tiles[blockIdx.x];
    for (int i = threadIdx.x; i < tile.count; i += blockDim.x)
        z_chunk[tok_t[tile.begin + i]] = z_wm[tile.wm_begin + i];
}

// Host streaming: the document of every token of a chunk, from the canonical token numbers, with one 16-byte
// look-up per token.  blocks[b] describes the canonical tokens 64 b .. 64 b + 63: .x = ordinal (among the non-empty
// documents) of the document that holds token 64 b, .y/.z = 64-bit mask whose bit j > 0 says that token 64 b + j is
// the first of its document.  The ordinal of token t's document is .x plus the mask bits up to t's own; ne_doc
// maps ordinals to document numbers when the corpus has empty documents (null: they are the same).
__global__ void expand_tok_doc_kernel(const uint32_t *__restrict__ tok_t, int64_t n, int64_t t0,
                                      const uint4 *__restrict__ blocks, const int32_t *__restrict__ ne_doc,
                                      int32_t *__restrict__ tok_doc) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        const int64_t t = t0 + (int64_t)tok_t[i];
        const uint4 q = blocks[t >> 6];
        const unsigned long long mask = (((unsigned long long)q.z << 32) | (unsigned long long)q.y) & (~0ull >> (63 - (int)(t & 63)));
        const int32_t ord = (int32_t)q.x + (int32_t)__popcll(mask);
        tok_doc[i] = ne_doc ? ne_doc[ord] : ord;
    }
}

// word-major copy of the assignments (after init / set_z; during iterations the E-step writes it)
template <typename ZT>
__global__ void fill_zwm_kernel(const Tile *tiles, const uint32_t *tok_t, const ZT *z, int64_t z_rel, ZT *z_wm) {
    const Tile tile = tiles[blockIdx.x];
    for (int i = threadIdx.x; i < tile.count; i += blockDim.x)
        z_wm[tile.wm_begin + i] = z[z_rel + (int64_t)tok_t[tile.begin + i]];
}

// ---------------------------------------------------------------------------------------------
// Block-wide exclusive scan of one uint32 per thread; returns the exclusive prefix, *total = block sum.
// scratch must hold blockDim.x/64 + 1 values.  Contains two __syncthreads() when the block has several wavefronts.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *scratch, uint32_t *total) {
    const int lane = lane_id(), wave = threadIdx.x / kWave, nwaves = (blockDim.x + kWave - 1) / kWave;
    const uint32_t incl = wave_incl_scan(v);
    if (blockDim.x <= kWave) {   // a single wavefront needs neither LDS nor barriers
        *total = readlane_u32(incl, kWave - 1);
        return incl - v;
    }
    if (lane == kWave - 1) scratch[wave] = incl;
    __syncthreads();
    uint32_t off = 0, tot = 0;
    for (int w = 0; w < nwaves; w++) { const uint32_t s = scratch[w]; if (w < wave) off += s; tot += s; }
    __syncthreads();
    *total = tot;
    return off + incl - v;
}

// ---------------------------------------------------------------------------------------------
// Segmented count of a short segment by one wavefront, in registers (bound by its vector instructions: 535,000 segments of
// 90 assignments take 0.21 ms, 0.23 with a compare and a selection per step and 21 steps for every segment; neither several segments per wavefront nor their loads ahead of time changed that):
// the sort-and-count of Sec. 3.3 taken
// literally.  Lane i holds assignment i (lanes past the end an all-ones key); a bitonic network of 21
// compare-exchange steps sorts the 64 keys (partners at lane ^ m: DPP quad permutations and row mirrors for m = 1,
// 2, 3, 7, 15, the LDS crossbar for the others; the lower lane of a pair keeps the smaller key).  A lane whose key
// differs from its left neighbour's starts a topic: the number of such lanes before it is the topic's slot in the
// row, the distance to the next such lane (both read off the wave-wide mask of these lanes) its count, and the
// lane stores the entry.  Segments of 65 to 128 assignments hold two keys per lane and add one merge stage.  About
// 90 vector instructions per segment (200 with two keys per lane) where the bitmap version below spends 390: it
// clears, scans and enumerates K / 32 bitmap words whatever the segment's length.
// ---------------------------------------------------------------------------------------------
// The lane keeps the middle one of its key, its partner's and a bound: 0 in the lower lane of a pair, which makes that the smaller key,
// all ones in the upper one (one instruction where a compare and a selection are two, and the masks are formed once per wavefront).
struct SortBounds { uint32_t b[6]; };   // by the bit of the lane number that tells upper from lower
__device__ __forceinline__ SortBounds sort_bounds(int lane) {
    SortBounds s;
#pragma unroll
    for (int i = 0; i < 6; i++) s.b[i] = (uint32_t)((int)((uint32_t)lane << (31 - i)) >> 31);
    return s;
}
__device__ __forceinline__ uint32_t middle_of(uint32_t a, uint32_t b, uint32_t c) {
    return max(min(a, b), min(max(a, b), c));   // (v_med3_u32)
}
template <int XOR>
__device__ __forceinline__ uint32_t sort_exchange(uint32_t v, int lane, const SortBounds &bounds) {
    uint32_t o;
    if (XOR == 1) o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);            // quad_perm [1,0,3,2]
    else if (XOR == 2) o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);       // quad_perm [2,3,0,1]
    else if (XOR == 3) o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x1B, 0xf, 0xf, true);       // quad_perm [3,2,1,0]
    else if (XOR == 7) o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);      // row_half_mirror
    else if (XOR == 15) o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true);     // row_mirror
    else if (XOR < 32) o = (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (XOR << 10) | 0x1f);   // lane ^ XOR inside 32 lanes
    else o = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ XOR) << 2, (int)v);
    constexpr int bit = XOR >= 32 ? 5 : XOR >= 16 ? 4 : XOR >= 8 ? 3 : XOR >= 4 ? 2 : XOR >= 2 ? 1 : 0;   // the highest one of XOR
    return middle_of(v, o, bounds.b[bit]);
}

// the 64 keys of one register, ascending over the lanes; len: no more than this many lanes, from the first on, hold anything but the
// largest key there is (16 keys take 10 of the 21 steps, 32 take 15)
__device__ __forceinline__ uint32_t sort64(uint32_t v, int lane, int len, const SortBounds &bounds) {
    auto step = [&](auto x) { v = sort_exchange<decltype(x)::value>(v, lane, bounds); };
    using std::integral_constant;
    step(integral_constant<int, 1>{});
    step(integral_constant<int, 3>{}); step(integral_constant<int, 1>{});
    step(integral_constant<int, 7>{}); step(integral_constant<int, 2>{}); step(integral_constant<int, 1>{});
    step(integral_constant<int, 15>{}); step(integral_constant<int, 4>{}); step(integral_constant<int, 2>{}); step(integral_constant<int, 1>{});
    if (len <= 16) return v;
    step(integral_constant<int, 31>{}); step(integral_constant<int, 8>{}); step(integral_constant<int, 4>{}); step(integral_constant<int, 2>{});
    step(integral_constant<int, 1>{});
    if (len <= 32) return v;
    step(integral_constant<int, 63>{}); step(integral_constant<int, 16>{}); step(integral_constant<int, 8>{}); step(integral_constant<int, 4>{});
    step(integral_constant<int, 2>{}); step(integral_constant<int, 1>{});
    return v;
}
// two ascending registers of 64 keys -> one ascending sequence of 128 (v0's lanes, then v1's): the last stage of the network
__device__ __forceinline__ void merge128(uint32_t &v0, uint32_t &v1, int lane, const SortBounds &bounds) {
    const uint32_t o1 = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 63) << 2, (int)v1);   // key 127 - i for key i
    const uint32_t o0 = (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ 63) << 2, (int)v0);
    v0 = min(v0, o1); v1 = max(v1, o0);
    auto step = [&](auto x) {
        v0 = sort_exchange<decltype(x)::value>(v0, lane, bounds);
        v1 = sort_exchange<decltype(x)::value>(v1, lane, bounds);
    };
    using std::integral_constant;
    step(integral_constant<int, 32>{}); step(integral_constant<int, 16>{}); step(integral_constant<int, 8>{});
    step(integral_constant<int, 4>{}); step(integral_constant<int, 2>{}); step(integral_constant<int, 1>{});
}

// R = 1: segments of at most 64 assignments; R = 2: of at most 128, two keys per lane (lane i holds keys i and 64 + i).
template <typename ZT, int R>
__device__ __forceinline__ void count_segment_wave(const ZT *__restrict__ zs, int len, uint2 *rec, uint32_t *__restrict__ row,
                                                   uint32_t count_bits) {
    const int lane = lane_id();
    constexpr uint32_t kNone = 0xffffffffu;
    uint32_t v0 = lane < len ? (uint32_t)zs[lane] : kNone;
    uint32_t v1 = R > 1 && lane + kWave < len ? (uint32_t)zs[lane + kWave] : kNone;
    const SortBounds bounds = sort_bounds(lane);
    v0 = sort64(v0, lane, R > 1 ? kWave : len, bounds);
    if (R > 1) { v1 = sort64(v1, lane, len - kWave, bounds); merge128(v0, v1, lane, bounds); }
    // the i-th smallest key now sits at position i (v0's lanes, then v1's); the all-ones keys follow the len real ones.
    // A key that differs from its left neighbour starts a topic: its slot in the row is the number of such keys
    // before it, its count the distance to the next one (or to the end of the segment).
    const uint32_t left0 = (uint32_t)__builtin_amdgcn_update_dpp((int)0xfffffffeu, (int)v0, 0x138, 0xf, 0xf, false);   // wave_shr:1
    const unsigned long long h0 = __builtin_amdgcn_ballot_w64(v0 != kNone && v0 != left0);
    unsigned long long h1 = 0ull;
    if (R > 1) {
        const uint32_t left1 = (uint32_t)__builtin_amdgcn_update_dpp((int)readlane_u32(v0, kWave - 1), (int)v1, 0x138, 0xf, 0xf, false);
        h1 = __builtin_amdgcn_ballot_w64(v1 != kNone && v1 != left1);
    }
    const int n0 = (int)__builtin_popcountll(h0), kd = n0 + (int)__builtin_popcountll(h1);
    const int after0 = h1 ? kWave + (int)__builtin_ctzll(h1) : len;        // first topic start behind v0's keys
    {
        const unsigned long long above = (h0 >> lane) >> 1;                // topic starts at the lanes above this one
        const int next = above ? lane + 1 + (int)__builtin_ctzll(above) : after0;
        const uint32_t slot = __builtin_amdgcn_mbcnt_hi((uint32_t)(h0 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h0, 0u));
        if (__builtin_amdgcn_inverse_ballot_w64(h0)) row[slot] = (v0 << count_bits) | (uint32_t)(next - lane);
    }
    if (R > 1 && h1) {
        const unsigned long long above = (h1 >> lane) >> 1;
        const int next = above ? lane + 1 + (int)__builtin_ctzll(above) : len - kWave;   // in v1's own numbering
        const uint32_t slot = (uint32_t)n0 + __builtin_amdgcn_mbcnt_hi((uint32_t)(h1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)h1, 0u));
        if (__builtin_amdgcn_inverse_ballot_w64(h1)) row[slot] = (v1 << count_bits) | (uint32_t)(next - lane);
    }
    // pad to the next multiple of 4 entries with (last topic, count 0), as the kernel below does
    const uint32_t last = R > 1 && len > kWave ? readlane_u32(v1, len - kWave - 1) : readlane_u32(v0, len - 1);
    if (lane < ((kd + 3) & ~3) - kd) row[kd + lane] = last << count_bits;
    if (lane == 0) rec->y = (uint32_t)kd;
}

// ---------------------------------------------------------------------------------------------
// CountByDZ (Alg. 1; the "segmented count" of Sec. 3.3), one workgroup per document (or light word: its row of B).
// The document's assignments are contiguous (z is kept in document order, so the "shuffle" of Sec. 3.3
// is the E-step's scattered store).  Instead of sorting, the workgroup marks the topics present in a
// K-bit LDS bitmap; popcount prefix sums over the bitmap give every present topic its rank, i.e. its
// slot in the ascending row; counts are accumulated per slot with LDS atomics.
// Rows whose K_d exceeds lds_entries are accumulated directly in the global row.
// ---------------------------------------------------------------------------------------------
// One grouping of the assignments: list[i] numbers the segments to count, segment s is z[ptr[s]..ptr[s+1]) with
// z[0] at position z_first of that numbering (a streaming buffer holds one chunk only); its row goes to ent from
// rec[s].x * 32 on, its length to rec[s].y.
struct SegGroup { const int32_t *list; const int64_t *ptr; const void *z; int64_t z_first; uint2 *rec; uint32_t *ent; };

// One segment of len > 0 assignments at zd by the whole workgroup, or (WAVE) by one wavefront of it; lds: bitmap, rank prefixes
// (nwords words each), lds_entries entries of the row; scan_scratch: a word per wavefront and one more.
template <typename ZT, bool WAVE = false>
__device__ __forceinline__ void count_segment_block(const ZT *__restrict__ zd, int len, uint2 *rec, uint32_t *__restrict__ row, uint32_t count_bits,
                                                    int nwords, int lds_entries, uint32_t *lds, uint32_t *scan_scratch) {
    const int tid = WAVE ? lane_id() : (int)threadIdx.x, nt = WAVE ? kWave : (int)blockDim.x;
    auto barrier = [] { if (WAVE) wave_lds_fence(); else __syncthreads(); };
    uint32_t *bitmap = lds;                // [nwords]
    uint32_t *wpre = lds + nwords;         // [nwords] exclusive popcount prefix
    uint32_t *ent_lds = wpre + nwords;     // [lds_entries]
    for (int w = tid; w < nwords; w += nt) bitmap[w] = 0u;
    barrier();
    for_each_z(zd, (int64_t)len, tid, nt, [&](uint32_t k) { atomicOr(&bitmap[k >> 5], 1u << (k & 31u)); });
    barrier();
    // ranks: exclusive prefix of popcounts over the bitmap words.  Every thread takes a contiguous piece of the
    // bitmap (ascending topics), so one scan over the threads' totals serves all words
    const int wpt = (nwords + nt - 1) / nt;
    const int wb = min(tid * wpt, nwords), we = min(wb + wpt, nwords);
    uint32_t mine = 0;
    for (int w = wb; w < we; w++) mine += (uint32_t)__popc(bitmap[w]);
    uint32_t total;
    uint32_t first;
    if (WAVE) {
        const uint32_t incl = wave_incl_scan(mine);
        total = readlane_u32(incl, kWave - 1);
        first = incl - mine;
    } else first = block_excl_scan(mine, scan_scratch, &total);
    const int kd = (int)total;
    const bool in_lds = kd <= lds_entries;
    uint32_t *ent = in_lds ? ent_lds : row;
    // slot r of the row starts as (topic, count 0): enumerate the set bits of the thread's words
    {
        uint32_t r = first;
        for (int w = wb; w < we; w++) {
            uint32_t m = bitmap[w];
            wpre[w] = r;
            while (m) { const int b = __ffs((int)m) - 1; m &= m - 1u; ent[r++] = (uint32_t)(w * 32 + b) << count_bits; }
        }
    }
    barrier();
    for_each_z(zd, (int64_t)len, tid, nt, [&](uint32_t k) {
        const uint32_t wd = bitmap[k >> 5];
        const uint32_t r = wpre[k >> 5] + (uint32_t)__popc(wd & ((1u << (k & 31u)) - 1u));
        atomicAdd(&ent[r], 1u);
    });
    barrier();
    if (in_lds)
        for (int r = tid; r < kd; r += nt) row[r] = ent_lds[r];
    // pad to the next multiple of 4 entries with (last topic, count 0): the sampler reads rows in 16-byte pieces,
    // and a draw that rounding pushes past the end of the row then still lands on the last topic
    if (tid < 4) {
        const int r = kd + tid;
        if (r < ((kd + 3) & ~3)) row[r] = ent[kd - 1] & ~((1u << count_bits) - 1u);
    }
    if (tid == 0) rec->y = (uint32_t)kd;
}

// The first na workgroups count the segments of group a, the others those of group b: documents and light words share a
// launch, which spares a small corpus two of them.
template <typename ZT>
__global__ void __launch_bounds__(1024) count_dz_kernel(SegGroup a, int64_t na, SegGroup b, uint32_t count_bits, int nwords,
                                                        int lds_entries) {
    extern __shared__ uint32_t lds_u32[];
    __shared__ uint32_t scan_scratch[20];
    const bool first_group = (int64_t)blockIdx.x < na;
    const SegGroup &g = first_group ? a : b;
    const int d = g.list[(int64_t)blockIdx.x - (first_group ? 0 : na)];
    const int64_t begin = g.ptr[d];
    const int len = (int)(g.ptr[d + 1] - begin);
    if (len == 0) { if (threadIdx.x == 0) g.rec[d].y = 0u; return; }
    const ZT *__restrict__ zd = reinterpret_cast<const ZT *>(g.z) + (begin - g.z_first);
    uint32_t *row = g.ent + (size_t)g.rec[d].x * 32u;
    if (blockDim.x == kWave && len <= 2 * kWave) {   // a short segment and a single wavefront: sorted in registers
        if (len <= kWave) count_segment_wave<ZT, 1>(zd, len, g.rec + d, row, count_bits);
        else count_segment_wave<ZT, 2>(zd, len, g.rec + d, row, count_bits);
        return;
    }
    count_segment_block(zd, len, g.rec + d, row, count_bits, nwords, lds_entries, lds_u32, scan_scratch);
}

// ---------------------------------------------------------------------------------------------
// Preprocess + BuildTree (Alg. 1; Eq. 2; Sec. 3.2.4), one workgroup of 256, 512 or 1,024 threads per dense row.
//   Bhat_vk  = (float(B_vk) + beta) / denom_k,  denom_k = float(C_k) + float(V) * beta   -- single-rounded fp32 ops
//   l3_64[i] = running sum of Bhat_v through topic (i+1)*64 - 1, accumulated in binary64
//   l3[i]    = round32(l3_64[i])                                           -- tree level above the bottom, W = 64
// Pad columns k in [K, Kpad) get Bhat = 0, so the last block's running sum is the row total.
// The bottom level (one prefix sum per topic) is not stored; the sampler rebuilds the 64 entries it needs.
// ---------------------------------------------------------------------------------------------
// Denominators of Eq. 2, one per topic: float(C_k) + float(V) * beta (the conversion rounds to nearest even).
// Pad columns get an infinite one, so that their Bhat comes out as zero.  The totals move from the accumulators, which are
// cleared for the next M-step, to their place of rest.
__global__ void denominators_kernel(unsigned long long *acc, unsigned long long *ck, float *denom, int K, int Kpad, float vbeta) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < K) {
        const unsigned long long c = acc[k];
        acc[k] = 0ull; ck[k] = c;
        denom[k] = (float)c + vbeta;
    } else if (k < Kpad) denom[k] = __builtin_inff();
}

// One dense row: its word (the tree levels are indexed by word) and its segment of the word-major assignments.  count >= 0:
// the workgroup histograms the segment in LDS, `range` topics at a time, and the counts never reach memory; count < 0: the
// word has too many tokens for one workgroup, its row of B was counted by count_slabs_kernel and is cleared here.
// The last row has no tokens: it yields the base vector (Bhat of a zero count) and its running sums for the light words.
//
// Bound by the store of Bhat, 4 Kpad bytes per row, and by the row's chain of steps.  Counting through memory (atomics into
// B, then read and clear it) moved three times that: K = 70,000, 4,002 rows of 375 tokens: 966 + 271 us before, 428 + 27 now
// (2.6 TB/s); K = 10,000, 1,450 rows: 44 + 66 us before, 43 + 41 now.  Barriers that wait for LDS only, a row's few assignments
// held in registers over the ranges and two steps per exchange of running sums (three do not leave two workgroups per CU
// their registers) took the 70,000-topic case from 740 us to 428.
// The running sums associate in groups of 1,024 columns whatever the workgroup's size.
struct PhiRow { int32_t word; int32_t count; int64_t begin; };
constexpr int kPhiSteps = 2;   // steps of 4 columns per thread that share one histogram and one exchange of running sums
constexpr int kPhiHeld = 4;    // assignments per thread that are read once and held

// Bhat of the n columns from r0 on of the row whose columns start at rbase, and the lanes' running sums over their wavefront's
// columns.  held: zr has the row's assignments.
template <typename ZT>
__device__ __forceinline__ void phi_range(const PhiRow pr, const ZT *__restrict__ zs, bool held, const uint32_t (&zr)[kPhiHeld], size_t rbase, int r0, int n,
                                          int32_t *cwk, const float *denom, float *phi, float beta, int4 *phi_hist4, double (&incl)[kPhiSteps]) {
    uint32_t *phi_hist = reinterpret_cast<uint32_t *>(phi_hist4);
    const int step = 4 * (int)blockDim.x;
    const bool own = pr.count >= 0;
    float4 den[kPhiSteps];             // requested before the counting
#pragma unroll
    for (int st = 0; st < kPhiSteps; st++) {
        const int k = st * step + (int)threadIdx.x * 4;
        den[st] = k < n ? *reinterpret_cast<const float4 *>(denom + r0 + k) : make_float4(1.f, 1.f, 1.f, 1.f);
    }
    if (own) {
        for (int k = threadIdx.x; k < n / 4; k += blockDim.x) phi_hist4[k] = make_int4(0, 0, 0, 0);
        lds_barrier();
        auto count = [&](uint32_t k) { if (k - (uint32_t)r0 < (uint32_t)n) atomicAdd(&phi_hist[k - (uint32_t)r0], 1u); };
        if (held) {
#pragma unroll
            for (int j = 0; j < kPhiHeld; j++) count(zr[j]);
        } else {
            block_for_each_z(zs, (int64_t)pr.count, count);
        }
        lds_barrier();
    }
#pragma unroll
    for (int st = 0; st < kPhiSteps; st++) {
        if (st * step >= n) break;     // uniform
        const int k = st * step + (int)threadIdx.x * 4;
        float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < n) {   // n is a multiple of 64, so k..k+3 are all inside the padded row
            int4 c;
            if (own) c = phi_hist4[k / 4];
            else c = *reinterpret_cast<const int4 *>(cwk + rbase + r0 + k);
            f.x = ((float)c.x + beta) / den[st].x; f.y = ((float)c.y + beta) / den[st].y;
            f.z = ((float)c.z + beta) / den[st].z; f.w = ((float)c.w + beta) / den[st].w;
            *reinterpret_cast<float4 *>(phi + rbase + r0 + k) = f;
            if (!own) *reinterpret_cast<int4 *>(cwk + rbase + r0 + k) = make_int4(0, 0, 0, 0);
        }
        incl[st] = wave_incl_scan((((double)f.x + (double)f.y) + (double)f.z) + (double)f.w);
    }
}
template <typename ZT>
__device__ __forceinline__ bool phi_hold(const PhiRow pr, const ZT *__restrict__ zs, uint32_t (&zr)[kPhiHeld]) {
    const bool held = pr.count >= 0 && pr.count <= kPhiHeld * (int)blockDim.x;
#pragma unroll
    for (int j = 0; j < kPhiHeld; j++) {
        const int i = (int)threadIdx.x + j * (int)blockDim.x;
        zr[j] = held && i < pr.count ? (uint32_t)zs[i] : 0xffffffffu;
    }
    return held;
}

template <typename ZT>
__device__ __forceinline__ void phi_row(const PhiRow pr, size_t row, const ZT *z_wm, int32_t *cwk, const float *denom, float *phi, float *l3,
                                        double *l3_64, float *sumphi, int Kpad, int n3, int n3pad, float beta, int range, int4 *phi_hist4) {
    __shared__ double wave_tot[kPhiSteps * 16];
    __shared__ float row_total;
    const int v = pr.word, step = 4 * (int)blockDim.x;
    const int lane = lane_id(), wave = threadIdx.x / kWave, nwaves = blockDim.x / kWave;
    const ZT *__restrict__ zs = z_wm + pr.begin;
    uint32_t zr[kPhiHeld];
    const bool held = phi_hold(pr, zs, zr);
    double carry = 0.0;
    for (int r0 = 0; r0 < Kpad; r0 += range) {
        const int n = min(range, Kpad - r0);
        double incl[kPhiSteps];
        phi_range(pr, zs, held, zr, row * (size_t)Kpad, r0, n, cwk, denom, phi, beta, phi_hist4, incl);
#pragma unroll
        for (int st = 0; st < kPhiSteps; st++)
            if (st * step < n && lane == kWave - 1) wave_tot[st * 16 + wave] = incl[st];
        lds_barrier();
#pragma unroll
        for (int st = 0; st < kPhiSteps; st++) {
            if (st * step >= n) break;
            double woff = 0.0, start = 0.0;    // `start`: running sum before the 1,024 columns of this wavefront
            for (int g = 0; g < nwaves; g += 4) {
                double btot = 0.0;
                if (g == (wave & ~3)) start = carry;
#pragma unroll
                for (int w = 0; w < 4; w++) {
                    const double tw = wave_tot[st * 16 + g + w];
                    if (g + w == wave) woff = btot;
                    btot += tw;
                }
                carry += btot;
            }
            const int k = st * step + (int)threadIdx.x * 4;
            if (k < n && ((k + 3) & (kWave - 1)) == kWave - 1) {
                const double run = start + woff + incl[st];       // running sum through topic r0 + k + 3, the end of a block
                const int i = (r0 + k + 3) / kWave;
                l3_64[(size_t)v * (size_t)n3 + (size_t)i] = run;
                l3[(size_t)v * (size_t)n3pad + (size_t)i] = (float)run;
                if (i == n3 - 1) row_total = (float)run;
            }
        }
        lds_barrier();
    }
    const float total = row_total;   // written before the loop's last barrier
    for (int i = n3 + (int)threadIdx.x; i < n3pad; i += blockDim.x) l3[(size_t)v * (size_t)n3pad + i] = total;
    if (threadIdx.x == 0) sumphi[v] = total;
}

// The same with a workgroup per `range` columns of a row, for few rows of many topics (bound by a row's chain of steps: 22 rows of
// 70,000 topics on 22 of 256 CUs took 53 us): first Bhat, and in l3_64 the running sums at
// the block ends inside each wavefront's 256 columns ...
template <typename ZT>
__device__ __forceinline__ void phi_part(const PhiRow pr, size_t row, int r0, const ZT *z_wm, int32_t *cwk, const float *denom, float *phi, double *l3_64,
                                         int Kpad, int n3, float beta, int range, int4 *phi_hist4) {
    const int n = min(range, Kpad - r0);
    const ZT *__restrict__ zs = z_wm + pr.begin;
    uint32_t zr[kPhiHeld];
    const bool held = phi_hold(pr, zs, zr);
    double incl[kPhiSteps];
    phi_range(pr, zs, held, zr, row * (size_t)Kpad, r0, n, cwk, denom, phi, beta, phi_hist4, incl);
#pragma unroll
    for (int st = 0; st < kPhiSteps; st++) {
        const int k = st * 4 * (int)blockDim.x + (int)threadIdx.x * 4;
        if (k < n && ((k + 3) & (kWave - 1)) == kWave - 1) l3_64[(size_t)pr.word * (size_t)n3 + (size_t)((r0 + k + 3) / kWave)] = incl[st];
    }
}
// ... then a workgroup per row adds what lies before: the same sums in the same order as phi_row's.  LDS: n3 doubles, one per 16 blocks.
// A group is 1,024 columns, 16 blocks, those of four wavefronts.
__global__ void __launch_bounds__(256) phi_sums_kernel(const PhiRow *rows, float *l3, double *l3_64, float *sumphi, int n3, int n3pad) {
    extern __shared__ double ps_lds[];
    const int ngroups = (n3 + 15) / 16;
    double *inside = ps_lds, *before = ps_lds + n3;   // sums inside a wavefront's columns; sum of a group, then of all before it
    const size_t v = (size_t)rows[blockIdx.x].word;
    for (int i = threadIdx.x; i < n3; i += blockDim.x) inside[i] = l3_64[v * (size_t)n3 + i];
    __syncthreads();
    auto wave_total = [&](int g, int w) {             // (the last wavefront with columns may have fewer than four blocks)
        const int first = 16 * g + 4 * w;
        return first < n3 ? inside[min(first + 3, n3 - 1)] : 0.0;
    };
    for (int g = threadIdx.x; g < ngroups; g += blockDim.x) {
        double sum = 0.0;
        for (int w = 0; w < 4; w++) sum += wave_total(g, w);
        before[g] = sum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double carry = 0.0;
        for (int g = 0; g < ngroups; g++) { const double sum = before[g]; before[g] = carry; carry += sum; }
    }
    __syncthreads();
    float last = 0.f;
    for (int i = threadIdx.x; i < n3; i += blockDim.x) {
        const int g = i / 16, wave = (i % 16) / 4;
        double woff = 0.0;
        for (int w = 0; w < wave; w++) woff += wave_total(g, w);
        const double run = before[g] + woff + inside[i];
        l3_64[v * (size_t)n3 + i] = run;
        l3[v * (size_t)n3pad + i] = (float)run;
        if (i == n3 - 1) { sumphi[v] = (float)run; last = (float)run; }
    }
    __shared__ float row_total;
    if ((int)threadIdx.x == (n3 - 1) % (int)blockDim.x) row_total = last;
    __syncthreads();
    for (int i = n3 + (int)threadIdx.x; i < n3pad; i += blockDim.x) l3[v * (size_t)n3pad + i] = row_total;
}

// PARTS: grid row y takes the y-th range of columns.
template <typename ZT, bool PARTS>
__global__ void __launch_bounds__(1024, 8) phi_tree_kernel(const PhiRow *rows, const ZT *z_wm, int32_t *cwk, const float *denom,
                                                        float *phi, float *l3, double *l3_64, float *sumphi, int Kpad,
                                                        int n3, int n3pad, float beta, int range) {
    extern __shared__ int4 phi_lds[];
    const PhiRow pr = rows[blockIdx.x];
    if (PARTS) phi_part(pr, (size_t)blockIdx.x, (int)blockIdx.y * range, z_wm, cwk, denom, phi, l3_64, Kpad, n3, beta, range, phi_lds);
    else phi_row(pr, (size_t)blockIdx.x, z_wm, cwk, denom, phi, l3, l3_64, sumphi, Kpad, n3, n3pad, beta, range, phi_lds);
}

// ---------------------------------------------------------------------------------------------
// Preprocess + BuildTree for the light words (one wavefront per word, or per W words of few tokens).  Their Bhat row is the base vector
// except at the word's non-zeros, so only those are evaluated (Eq. 2, same three binary32 operations) and
// stored next to the entries.  The running sums at the block ends follow from the base vector's running sums
// plus the cumulative difference (Bhat - base) of the non-zeros up to each block, all in binary64: the same
// sum of the same binary32 numbers as for a dense row, associated differently.
// LDS: a zero and the cumulative differences at the last non-zero of each block that has one, then a bit per block that has.
// ---------------------------------------------------------------------------------------------
struct LightParams {
    const int32_t *light_words; const uint2 *wrec; const uint32_t *lw_ent; float *lw_phi;
    const float *denom, *base; const double *basecum; float *l3; double *l3_64; float *sumphi;
    int n3, n3pad, n_light, n_wide;   // the first n_wide words have many tokens and a wavefront each
    uint32_t count_bits; float beta;
};
__host__ __device__ inline size_t light_lds_bytes(int n3) { return ((size_t)n3 + 1u + (size_t)(n3 + 63) / 64u) * 8u; }

// Up to W light words, numbers `first` to `end`, by one wavefront with light_lds_bytes(n3) of LDS at lds_dcum.  Bound by the chain of
// loads that leads to a word's non-zeros' denominators - its record, its entries, their denominators - where rows are short: the
// words of a wavefront take each of the three steps together (see words_per_wave() on the host).  A block's running sum needs the
// difference at the last block with a non-zero up to it, which is found by counting these (15 vector instructions per 64 blocks; by a
// running maximum over the lanes and differences stored by block 30: T = 36 M, K = 5,000 82 -> 79 us).
template <int W>
__device__ __forceinline__ void light_words(const LightParams &p, int first, int end, double *lds_dcum) {
    const int n3 = p.n3, n3pad = p.n3pad, lane = lane_id();
    const uint32_t count_bits = p.count_bits, cmask = (1u << count_bits) - 1u;
    const float beta = p.beta;
    const float *__restrict__ denom = p.denom, *__restrict__ base = p.base;
    const double *__restrict__ basecum = p.basecum;
    float *l3 = p.l3, *sumphi = p.sumphi;
    double *l3_64 = p.l3_64;
    uint32_t *has = reinterpret_cast<uint32_t *>(lds_dcum + n3 + 1);
    int word[W];
    uint2 rec[W];
#pragma unroll
    for (int w = 0; w < W; w++) {
        const int li = min(first + w, end - 1);
        word[w] = p.light_words[li]; rec[w] = p.wrec[li];
    }
    // the base vector's running sums of the first steps, requested under that chain
    constexpr int kSteps = 4;
    double cum[kSteps];
#pragma unroll
    for (int st = 0; st < kSteps; st++) cum[st] = basecum[min(st * kWave + lane, n3 - 1)];
    uint32_t e0[W];
    const int others = end - first > 1 ? kWave : 0;   // (a word that is alone: nothing is loaded in the others' place)
    float den0[W], base0[W];
#pragma unroll
    for (int w = 0; w < W; w++) e0[w] = lane < (w ? min((int)rec[w].y, others) : (int)rec[w].y) ? p.lw_ent[(size_t)rec[w].x * 32u + (size_t)lane] : 0u;
#pragma unroll
    for (int w = 0; w < W; w++) { den0[w] = denom[e0[w] >> count_bits]; base0[w] = base[e0[w] >> count_bits]; }
#pragma unroll
    for (int w = 0; w < W; w++) {
        if (first + w >= end) break;   // uniform
        const int v = word[w], nnz = (int)rec[w].y;
        const uint32_t *__restrict__ ent = p.lw_ent + (size_t)rec[w].x * 32u;
        float *__restrict__ val = p.lw_phi + (size_t)rec[w].x * 32u;
        for (int i = lane; i < (n3 + 63) / 64 * 2; i += kWave) has[i] = 0u;
        if (lane == 0) lds_dcum[0] = 0.0;
        wave_lds_fence();
        double carry = 0.0;
        int blocks = 0;                    // with a non-zero so far
        for (int j0 = 0; j0 < nnz; j0 += kWave) {
            const int j = j0 + lane;
            const bool valid = j < nnz;
            const uint32_t e = j0 == 0 ? e0[w] : valid ? ent[j] : 0u;
            const uint32_t k = e >> count_bits;
            double delta = 0.0;
            if (valid) {
                const float f = ((float)(e & cmask) + beta) / (j0 == 0 ? den0[w] : denom[k]);
                val[j] = f;
                delta = (double)f - (double)(j0 == 0 ? base0[w] : base[k]);
            }
            const double incl = wave_incl_scan(delta) + carry;
            const int blk = (int)(k >> 6);
            int next_blk = __builtin_amdgcn_update_dpp(-1, blk, 0x130, 0xf, 0xf, false);   // wave_shl:1
            if (j0 + kWave < nnz && lane == kWave - 1) next_blk = (int)((ent[j + 1] >> count_bits) >> 6);
            const unsigned long long ends = __builtin_amdgcn_ballot_w64(valid && (j + 1 == nnz || blk != next_blk));
            if (__builtin_amdgcn_inverse_ballot_w64(ends)) {
                lds_dcum[blocks + (int)bits_up_to_lane(ends)] = incl;
                atomicOr(&has[blk >> 5], 1u << (blk & 31));
            }
            blocks += (int)__builtin_popcountll(ends);
            carry = readlane_f64(incl, 63);
        }
        wave_lds_fence();
        // A block's difference is that of the last block with a non-zero up to it: the blocks with one are counted.
        int before = 0;
        float total = 0.f;
        for (int i0 = 0; i0 < n3; i0 += kSteps * kWave) {
#pragma unroll
            for (int st = 0; st < kSteps; st++) {
                if (i0 + st * kWave >= n3) break;   // uniform
                const int i = i0 + st * kWave + lane;
                const uint2 m = reinterpret_cast<const uint2 *>(has)[i0 / kWave + st];
                const unsigned long long mask = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)m.y) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)m.x);
                const double delta = lds_dcum[before + (int)bits_up_to_lane(mask)];
                before += (int)__builtin_popcountll(mask);
                if (i < n3) {
                    const double run = (i0 ? basecum[i] : cum[st]) + delta;
                    l3_64[(size_t)v * (size_t)n3 + (size_t)i] = run;
                    l3[(size_t)v * (size_t)n3pad + (size_t)i] = (float)run;
                    if (i == n3 - 1) total = (float)run;
                }
            }
        }
        wave_lds_fence();
        total = readlane_f32(total, (n3 - 1) & (kWave - 1));
        for (int i = n3 + lane; i < n3pad; i += kWave) l3[(size_t)v * (size_t)n3pad + i] = total;
        if (lane == 0) sumphi[v] = total;
    }
}

// The share of wavefront number `wave`: one of the first n_wide words, or W of the others.
template <int W>
__device__ __forceinline__ void light_share(const LightParams &p, int wave, double *lds_dcum) {
    const int first = W == 1 ? wave : min(wave, p.n_wide) + max(wave - p.n_wide, 0) * W;
    light_words<W>(p, first, W == 1 || wave < p.n_wide ? first + 1 : min(first + W, p.n_light), lds_dcum);
}
template <int W>
__global__ void __launch_bounds__(64) light_tree_kernel(LightParams p) {
    extern __shared__ double lds_dcum[];
    light_share<W>(p, (int)blockIdx.x, lds_dcum);
}

// Bhat rows of the words asked for, out[i][k], one workgroup each: a dense row is copied, a light word's is the base vector
// overwritten at its non-zeros.  rows[i] is the word's dense row, or -1 - its index among the light words.
// (One launch and one wait for all words: a copy or a launch, and two waits, per word took 6.4 ms for 400 words at K = 1,500.)
__global__ void __launch_bounds__(256) phi_export_kernel(const int32_t *rows, const float *phi, const float *base, const uint2 *wrec,
                                                         const uint32_t *lw_ent, const float *lw_phi, int K, int Kpad,
                                                         uint32_t count_bits, float *out) {
    const int row = rows[blockIdx.x];
    const float *__restrict__ src = row >= 0 ? phi + (size_t)row * (size_t)Kpad : base;
    float *__restrict__ dst = out + (size_t)blockIdx.x * (size_t)K;
    for (int k = threadIdx.x; k < K; k += blockDim.x) dst[k] = src[k];
    if (row >= 0) return;
    __syncthreads();
    const uint2 wr = wrec[-row - 1];
    for (int j = threadIdx.x; j < (int)wr.y; j += blockDim.x) dst[lw_ent[(size_t)wr.x * 32u + j] >> count_bits] = lw_phi[(size_t)wr.x * 32u + j];
}

// Statistics for the bandwidth model (exact in binary64 below 2^53), added to out[0..4]: the dense-branch counter slots
// (n_slots of them, by workgroup 0); nnz(A); sum_d K_d * L_d (row entries touched if every token read its row);
// sum_d K_d * U_d, U_d = distinct words of document d inside its chunk (row entries the sampler has to fetch: consecutive
// tokens of one (word, document) pair share the row); non-zeros of the sparse rows of B (what the next E-step stages for
// the light words).  A workgroup ends with one atomic per sum: a few hundred of them, since they are all to the same
// addresses (1,024 took 15 us).
struct StatsParams {
    const unsigned long long *slots; int n_slots;
    const uint2 *docrec; const int64_t *doc_ptr; const uint32_t *doc_words; int64_t D;
    const uint2 *wrec; int n_light; unsigned long long *out;
};

// the share of workgroup `block` of `nblocks`
__device__ __forceinline__ void stats_share(const StatsParams &p, int block, int nblocks) {
    double sums[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const int64_t first = (int64_t)block * blockDim.x + threadIdx.x, stride = (int64_t)nblocks * blockDim.x;
    if (block == 0)
        for (int i = threadIdx.x; i < p.n_slots; i += blockDim.x) sums[0] += (double)p.slots[i];
    for (int64_t d = first; d < p.D; d += stride) {
        const double kd = (double)p.docrec[d].y;
        sums[1] += kd; sums[2] += kd * (double)(p.doc_ptr[d + 1] - p.doc_ptr[d]); sums[3] += kd * (double)p.doc_words[d];
    }
    for (int64_t i = first; i < p.n_light; i += stride) sums[4] += (double)p.wrec[i].y;
    __shared__ double part[5][16];
#pragma unroll
    for (int q = 0; q < 5; q++) {
        const double w = readlane_f64(wave_incl_scan(sums[q]), 63);
        if (lane_id() == 0) part[q][threadIdx.x / kWave] = w;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        double sum = 0.0;
        for (int w = 0; w < (int)(blockDim.x / kWave); w++) sum += part[threadIdx.x][w];
        if (sum > 0.0) atomicAdd(&p.out[threadIdx.x], (unsigned long long)sum);
    }
}
__global__ void __launch_bounds__(256) stats_kernel(StatsParams p) { stats_share(p, (int)blockIdx.x, (int)gridDim.x); }

// ---------------------------------------------------------------------------------------------
// The M-step of a small corpus (16-bit assignments, some words light) in two launches.  A launch behind another costs 4.5 us whatever it does, and six or seven of
// them were half of an iteration at T = 100 K, K = 100, a quarter at T = 2.3 M, K = 777.
//
// First everything that counts: shares of the topic totals, slabs of the longest dense rows and long segments (documents and
// light words), a workgroup each, and the shorter segments, a wavefront each.  The workgroup that finishes the
// last share of the totals - it draws the last ticket, after its additions have reached memory - forms the denominators and
// the base vector with its running sums, under the rest of the launch.  Shares come first in the grid for that.
// ---------------------------------------------------------------------------------------------
struct MCounts {
    SegGroup docs, words;                   // (list: of the long segments)
    const int32_t *short_docs, *short_words;
    int n_tot, n_items, n_long_docs, n_long_words, n_short_docs, n_short_words;
    int64_t T, per_block;
    unsigned long long *acc, *ck;           // accumulators of the totals (zero again at the end), totals
    unsigned *ticket;                       // zero before and after
    const VzItem *items; int32_t *cwk;
    uint32_t count_bits; int nwords, lds_entries, wave_entries;   // entries of a row in LDS: of a workgroup, of a wavefront
    float vbeta, beta, *denom, *phi, *l3, *sumphi; double *l3_64;
    int K, Kpad, n3, n3pad, range, base_row, base_word;
};

__global__ void __launch_bounds__(256, 8) mstep_counts_kernel(MCounts p) {
    extern __shared__ int4 mc_lds4[];
    uint32_t *lds = reinterpret_cast<uint32_t *>(mc_lds4);
    __shared__ uint32_t scan_scratch[20];
    const uint16_t *z = reinterpret_cast<const uint16_t *>(p.docs.z), *z_wm = reinterpret_cast<const uint16_t *>(p.words.z);
    int b = (int)blockIdx.x;
    if (b < p.n_tot) {
        const int64_t first = (int64_t)b * p.per_block;
        count_slab(z + first, min(p.per_block, p.T - first), lds, 0, p.K, true, [&](int k, uint32_t h) { atomicAdd(&p.acc[k], (unsigned long long)h); });
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) scan_scratch[0] = atomicAdd(p.ticket, 1u);
        __syncthreads();
        if (scan_scratch[0] != (uint32_t)p.n_tot - 1u) return;
        __threadfence();
        if (threadIdx.x == 0) *p.ticket = 0u;
        for (int k = threadIdx.x; k < p.Kpad; k += blockDim.x) {   // (pad columns: Bhat comes out as zero)
            float d = __builtin_inff();
            if (k < p.K) {
                const unsigned long long c = __hip_atomic_load(&p.acc[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                p.acc[k] = 0ull; p.ck[k] = c;
                d = (float)c + p.vbeta;
            }
            p.denom[k] = d;
        }
        __syncthreads();
        phi_row(PhiRow{p.base_word, 0, 0}, (size_t)p.base_row, z_wm, p.cwk, p.denom, p.phi, p.l3, p.l3_64, p.sumphi, p.Kpad, p.n3, p.n3pad, p.beta,
                p.range, mc_lds4);
        return;
    }
    b -= p.n_tot;
    if (b < p.n_items) {
        const VzItem it = p.items[b];
        int32_t *row = p.cwk + (size_t)it.row * (size_t)p.Kpad;
        count_slab(z_wm + it.begin, (int64_t)it.count, lds, 0, p.K, true, [&](int k, uint32_t h) { atomicAdd(&row[k], (int)h); });
        return;
    }
    b -= p.n_items;
    const int n_long = p.n_long_docs + p.n_long_words;
    const bool whole = b < n_long;         // the workgroup's own segment, or one per wavefront
    const int nw = (int)(blockDim.x / kWave);
    int i = whole ? b : (b - n_long) * nw + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int n_docs = whole ? p.n_long_docs : p.n_short_docs, n_words = whole ? p.n_long_words : p.n_short_words;
    if (i >= n_docs + n_words) return;
    const bool doc = i < n_docs;
    const SegGroup &g = doc ? p.docs : p.words;
    const int32_t *list = whole ? g.list : doc ? p.short_docs : p.short_words;
    const int d = list[doc ? i : i - n_docs];
    const int64_t begin = g.ptr[d];
    const int len = (int)(g.ptr[d + 1] - begin);
    const uint16_t *zd = (doc ? z : z_wm) + begin;
    uint32_t *row = g.ent + (size_t)g.rec[d].x * 32u;
    if (whole) count_segment_block(zd, len, g.rec + d, row, p.count_bits, p.nwords, p.lds_entries, lds, scan_scratch);
    else if (len > 2 * kWave) {
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
        count_segment_block<uint16_t, true>(zd, len, g.rec + d, row, p.count_bits, p.nwords, p.wave_entries,
                                            lds + wave * (2 * p.nwords + p.wave_entries), nullptr);
    } else if (len > kWave) count_segment_wave<uint16_t, 2>(zd, len, g.rec + d, row, p.count_bits);
    else if (len > 0) count_segment_wave<uint16_t, 1>(zd, len, g.rec + d, row, p.count_bits);
    else if (lane_id() == 0) g.rec[d].y = 0u;
}

// Then everything that follows from the counts: dense rows of Bhat, a workgroup each, the statistics, and the light words, a wavefront
// each or W to a wavefront.
template <int W>
__global__ void __launch_bounds__(1024, 8) mstep_rows_kernel(const PhiRow *rows, int n_rows, const uint16_t *z_wm, int32_t *cwk, float *phi, int Kpad,
                                                             int range, StatsParams st, int n_stats, LightParams lp) {
    extern __shared__ int4 mr_lds4[];
    int b = (int)blockIdx.x;
    if (b < n_stats) { stats_share(st, b, n_stats); return; }
    b -= n_stats;
    if (b < n_rows) {
        phi_row(rows[b], (size_t)b, z_wm, cwk, lp.denom, phi, lp.l3, lp.l3_64, lp.sumphi, Kpad, lp.n3, lp.n3pad, lp.beta, range, mr_lds4);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), share = (b - n_rows) * (int)(blockDim.x / kWave) + wave;
    if (share < lp.n_wide + (lp.n_light - lp.n_wide + W - 1) / W)
        light_share<W>(lp, share, reinterpret_cast<double *>(reinterpret_cast<char *>(mr_lds4) + (size_t)wave * light_lds_bytes(lp.n3)));
}

// ---------------------------------------------------------------------------------------------
// Log-likelihood reduction (the per-token log-likelihood is the quality metric of Sec. 4): binary64 sums in a
// fixed order, so the result is the same in every run.  kReduceBlocks workgroups of kReduceThreads threads: thread
// i of workgroup b adds the elements b * kReduceThreads + i, + kReduceBlocks * kReduceThreads, ...; lanes are
// combined by a DPP scan, wavefronts and workgroups in index order.
// ---------------------------------------------------------------------------------------------
constexpr int kReduceBlocks = 256, kReduceThreads = 256;

__device__ __forceinline__ double block_sum_f64(double v, double *wave_part) {
    const double w = readlane_f64(wave_incl_scan(v), 63);
    if (lane_id() == 0) wave_part[threadIdx.x / kWave] = w;
    __syncthreads();
    double sum = 0.0;
    for (int i = 0; i < (int)(blockDim.x / kWave); i++) sum += wave_part[i];
    __syncthreads();
    return sum;
}

// block_part[b] = sum of workgroup b's share of in[0..n)
__global__ void __launch_bounds__(kReduceThreads) reduce_partials_kernel(const double *in, int64_t n, double *block_part) {
    __shared__ double wave_part[kReduceThreads / kWave];
    double v = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; i < n; i += (int64_t)kReduceBlocks * kReduceThreads) v += in[i];
    const double sum = block_sum_f64(v, wave_part);
    if (threadIdx.x == 0) block_part[blockIdx.x] = sum;
}

// block_part[b] = workgroup b's share of sum_d w_d ln(len_d + K alpha), w_d = wptr[d+1] - wptr[d] and
// len_d = lptr[d+1] - lptr[d]: the normaliser of theta_d, once per token that is scored in document d.
__global__ void __launch_bounds__(kReduceThreads) doc_norm_kernel(const int64_t *wptr, const int64_t *lptr, int64_t D,
                                                                   double k_alpha, double *block_part) {
    __shared__ double wave_part[kReduceThreads / kWave];
    double v = 0.0;
    for (int64_t d = (int64_t)blockIdx.x * kReduceThreads + threadIdx.x; d < D; d += (int64_t)kReduceBlocks * kReduceThreads) {
        const int64_t w = wptr[d + 1] - wptr[d];
        if (w > 0) v += (double)w * log((double)(lptr[d + 1] - lptr[d]) + k_alpha);
    }
    const double sum = block_sum_f64(v, wave_part);
    if (threadIdx.x == 0) block_part[blockIdx.x] = sum;
}

// *acc = (add ? *acc : 0) + sum of block_part[0..kReduceBlocks); one workgroup
__global__ void __launch_bounds__(kReduceThreads) reduce_final_kernel(const double *block_part, double *acc, int add) {
    __shared__ double wave_part[kReduceThreads / kWave];
    const double sum = block_sum_f64(threadIdx.x < kReduceBlocks ? block_part[threadIdx.x] : 0.0, wave_part);
    if (threadIdx.x == 0) *acc = (add ? *acc : 0.0) + sum;
}

// *out = (*sum_ln - *norm) / tokens: the per-token log-likelihood
__global__ void loglik_finish_kernel(const double *sum_ln, const double *norm, double tokens, double *out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *out = (*sum_ln - *norm) / tokens;
}

// Plain streaming copy (16 bytes per lane per step): the yardstick for achievable HBM bandwidth and the
// calibration kernel for the profiler's FETCH_SIZE / WRITE_SIZE counters.
__global__ void copy_probe_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n16) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n16; i += stride) dst[i] = src[i];
}

}  // namespace saber
