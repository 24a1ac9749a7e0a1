// Per-sample attention over the low-rank coordinates (section "Residual DCN",
// second paragraph: value/query/key copies of the low-rank map, an attention
// score matrix inserted between the low-rank maps, a temperature, and a skip
// connection).
//
// For one sample, the r low-rank coordinates are r scalar tokens:
//   S_ij = q_i k_j / tau,  A = softmax over j,  o = A v,  h = beta v + alpha o.
// A is never stored. Because S_ij = q_i k_j / tau is linear in k_j, the row
// maximum is q_i max_j k_j / tau when q_i >= 0 and q_i min_j k_j / tau
// otherwise (rounded multiplication is monotone, so the same holds in float),
// which removes the usual online-softmax rescaling: every exponent is
// exp2(c_i k_j - c_i k*_i) <= 1 with c_i = q_i log2(e) / tau.
//
// Float models: one workgroup per sample; k and v (and, in the backward column pass, the
// per-row coefficients) are staged in LDS as floats and read as broadcasts. bf16 models:
// the matrix-core kernels below.
#include <type_traits>

#include "device_common.h"
#include "kernels.h"

namespace rdcn {

namespace {

constexpr float LOG2E = 1.4426950408889634f;

__device__ __forceinline__ void block_minmax(float lo, float hi, float* red, float& out_lo, float& out_hi) {
    // wave reduction then across waves (blockDim <= 1024)
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
    if (lane == 0) {
        red[wave] = lo;
        red[16 + wave] = hi;
    }
    __syncthreads();
    lo = red[0];
    hi = red[16];
    for (int w = 1; w < nw; ++w) {
        lo = fminf(lo, red[w]);
        hi = fmaxf(hi, red[16 + w]);
    }
    out_lo = lo;
    out_hi = hi;
}

// Forward. P = [v | q | k] per sample in float (row stride ldp), h out (row stride ldh).
template <typename T>
__global__ __launch_bounds__(256) void k_attn_fwd(int64_t B, int r, float alpha, float beta, float inv_tau,
                                                 const float* __restrict__ P, int64_t ldp, T* __restrict__ H,
                                                 T* __restrict__ H2, int64_t ldh) {
    extern __shared__ float smem[];
    float* sk = smem;          // [r]
    float* sv = smem + r;      // [r]
    float* red = smem + 2 * r; // [32]
    const int64_t b = blockIdx.x;
    const float* pv = P + b * ldp;
    const float* pq = pv + r;
    const float* pk = pv + 2 * r;
    float lo = INFINITY, hi = -INFINITY;
    for (int j = threadIdx.x; j < r; j += blockDim.x) {
        const float kj = pk[j];
        sk[j] = kj;
        sv[j] = pv[j];
        lo = fminf(lo, kj);
        hi = fmaxf(hi, kj);
    }
    float kmin, kmax;
    block_minmax(lo, hi, red, kmin, kmax);  // includes a barrier after sk/sv are written
    for (int i = threadIdx.x; i < r; i += blockDim.x) {
        const float c = pq[i] * (LOG2E * inv_tau);
        const float mneg = -(c * (c >= 0.f ? kmax : kmin));
        float z0 = 0.f, z1 = 0.f, s0 = 0.f, s1 = 0.f;
        int j = 0;
        for (; j + 1 < r; j += 2) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(c, sk[j], mneg));
            const float e1 = __builtin_amdgcn_exp2f(fmaf(c, sk[j + 1], mneg));
            z0 += e0;
            z1 += e1;
            s0 = fmaf(e0, sv[j], s0);
            s1 = fmaf(e1, sv[j + 1], s1);
        }
        if (j < r) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(c, sk[j], mneg));
            z0 += e0;
            s0 = fmaf(e0, sv[j], s0);
        }
        const float o = (s0 + s1) / (z0 + z1);
        const float hv = beta * sv[i] + alpha * o;
        st<T>::store(H + b * ldh + i, hv);
        if (H2) st<T>::store(H2 + b * ldh + i, hv - st<T>::load(H + b * ldh + i));  // lo part of a hi + lo pair
    }
}

// Backward. gh = dLoss/dh (float, row stride ldg). Writes gP = [gv | gq | gk].
//   row pass (thread per query i):   Z_i = sum_j e_ij, o_i = sum_j e_ij v_j / Z_i,
//       gq_i = go_i/(Z_i tau) * (sum_j e_ij v_j k_j - o_i sum_j e_ij k_j),  go = alpha gh
//   column pass (thread per key j):  with a_i = go_i q_i/(Z_i tau), b_i = a_i o_i, c_i = go_i / Z_i
//       gk_j = v_j sum_i e_ij a_i - sum_i e_ij b_i,   gv_j = beta gh_j + sum_i e_ij c_i
// e_ij = exp2(c'_i k_j - c'_i k*_i) is recomputed identically in both passes.
template <typename T>
__global__ __launch_bounds__(256) void k_attn_bwd(int64_t B, int r, float alpha, float beta, float inv_tau,
                                                 const float* __restrict__ P, int64_t ldp, const float* __restrict__ GH,
                                                 int64_t ldg, T* __restrict__ GP, int64_t ldgp) {
    extern __shared__ float smem[];
    float* sk = smem;
    float* sv = smem + r;
    float* sc = smem + 2 * r;   // c'_i
    float* sm = smem + 3 * r;   // -c'_i k*_i
    float* sa = smem + 4 * r;   // a_i
    float* sb = smem + 5 * r;   // b_i
    float* sg = smem + 6 * r;   // c_i = go_i / Z_i
    float* red = smem + 7 * r;  // [32]
    const int64_t b = blockIdx.x;
    const float* pv = P + b * ldp;
    const float* pq = pv + r;
    const float* pk = pv + 2 * r;
    const float* gh = GH + b * ldg;
    T* gv_out = GP + b * ldgp;
    T* gq_out = gv_out + r;
    T* gk_out = gv_out + 2 * r;
    float lo = INFINITY, hi = -INFINITY;
    for (int j = threadIdx.x; j < r; j += blockDim.x) {
        const float kj = pk[j];
        sk[j] = kj;
        sv[j] = pv[j];
        lo = fminf(lo, kj);
        hi = fmaxf(hi, kj);
    }
    float kmin, kmax;
    block_minmax(lo, hi, red, kmin, kmax);
    for (int i = threadIdx.x; i < r; i += blockDim.x) {
        const float q = pq[i];
        const float c = q * (LOG2E * inv_tau);
        const float mneg = -(c * (c >= 0.f ? kmax : kmin));
        float z = 0.f, s = 0.f, w1 = 0.f, w2 = 0.f;
        for (int j = 0; j < r; ++j) {
            const float e = __builtin_amdgcn_exp2f(fmaf(c, sk[j], mneg));
            const float kj = sk[j];
            const float ev = e * sv[j];
            z += e;
            s += ev;
            w1 = fmaf(ev, kj, w1);
            w2 = fmaf(e, kj, w2);
        }
        const float rz = 1.0f / z;
        const float o = s * rz;
        const float go = alpha * gh[i];
        const float a = go * q * rz * inv_tau;
        st<T>::store(gq_out + i, go * rz * inv_tau * (w1 - o * w2));
        sc[i] = c;
        sm[i] = mneg;
        sa[i] = a;
        sb[i] = a * o;
        sg[i] = go * rz;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < r; j += blockDim.x) {
        const float kj = sk[j];
        float c1 = 0.f, c2 = 0.f, c3 = 0.f;
        for (int i = 0; i < r; ++i) {
            const float e = __builtin_amdgcn_exp2f(fmaf(sc[i], kj, sm[i]));
            c1 = fmaf(e, sa[i], c1);
            c2 = fmaf(e, sb[i], c2);
            c3 = fmaf(e, sg[i], c3);
        }
        st<T>::store(gk_out + j, sv[j] * c1 - c2);
        st<T>::store(gv_out + j, beta * gh[j] + c3);
    }
}

// ---------------------------------------------------------------------------
// bf16 models: the exponentials are computed on the vector ALU, every weighted
// sum over them runs on the matrix cores. Two forms, chosen per sample by its range of
// scores: panel sums (further down) and direct sums, one exponential per (row, key).
//
// Direct sums. For a 32-row x 32-key block of one
// sample, one v_mfma_f32_32x32x8_f16 leaves each lane 16 values e_ij of its row
// i = lane % 32, 8 of which form the B operand of a v_mfma_f32_16x16x32_f16 with
// K running over 16 keys (rows n and n + 16 share its columns and go to output
// slots 0-7 and 8-15; the A operand is zero in the other half); the A operand is a small
// per-sample matrix X^T whose rows are the quantities summed against e (v, 1,
// v k, k), each stored as an f16 hi + lo pair scaled by a power of two so the
// pair keeps about 21 significant bits. e itself is rounded to f16 (relative
// 2^-11); all sums of one row use the same rounded e, so the normalisation by Z
// is consistent. Output lane l holds quantities 4 (l / 16 % 2) .. +3 of row
// l % 16 (+16 for l >= 32).
//
// In the forward one wave owns up to ATT_NT 16-row tiles of one sample and loops
// over all keys, so row sums never leave its registers; a sample with more rows
// is split over W = ceil(tiles / ATT_NT) waves of one workgroup, which share the
// sample's keys and X^T in LDS.
//
// The forward saves each row's o_i and Z_i and, from the same MFMAs (four more
// rows of X^T), the one value D_i the query gradient needs. The backward is then
// left with column sums only (over rows, weighted by per-row coefficients that
// depend on o_i and Z_i): it computes the exponent arguments with the forward's
// product transposed (row records as the A operand, key fragments as B), which
// hands every lane the e values of one key for 16 rows: B operands with K
// running over rows. No e_ij is stored or exchanged between lanes.
// ---------------------------------------------------------------------------
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
#define LDS_AS __attribute__((address_space(3)))

constexpr int ATT_NT = 16;  // 16-row tiles per wave
// 16-key tiles the backward's direct sums carry through one pass over a sample's rows: four
// (the row records and Y^T fragment read per 32-row block serve 64 keys; eight spill at four
// waves per SIMD), eight in the kernels that also hold the panel sums, which run three
// (rank 256: 42.1 -> 38.5 us).
constexpr int ATT_BWD_KT = 4;
constexpr int ATT_BWD_KT_WIDE = 8;

__device__ __forceinline__ uint32_t pk_f16(float a, float b) {
    const f16x2_t v = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, v);
}

// power of two >= |m| (1 for m == 0), so x / scale lies in [-1, 1]
__device__ __forceinline__ float pow2_ceil(float m) {
    if (!(m > 0.f)) return 1.f;
    int e;
    const float f = frexpf(m, &e);  // m = f * 2^e, f in [0.5, 1)
    (void)f;
    return ldexpf(1.f, e);
}

// A wave-uniform float (the same value in every lane) moved to a scalar register.
__device__ __forceinline__ float uniform_f(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// Maximum / minimum over the wave, in every lane: row shifts and broadcasts by DPP (lane 63
// ends up with all 64 values; a shift's missing source leaves the lane's own value), one
// scalar read instead of six LDS-latency shuffles.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_f(float x) {
    const int v = __builtin_bit_cast(int, x);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_f<0x111, 0xf>(x));  // row_shr:1
    x = fmaxf(x, dpp_f<0x112, 0xf>(x));  // row_shr:2
    x = fmaxf(x, dpp_f<0x114, 0xf>(x));  // row_shr:4
    x = fmaxf(x, dpp_f<0x118, 0xf>(x));  // row_shr:8
    x = fmaxf(x, dpp_f<0x142, 0xa>(x));  // row_bcast:15 into rows 1 and 3
    x = fmaxf(x, dpp_f<0x143, 0xc>(x));  // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), 63));
}
__device__ __forceinline__ float wave_min(float x) { return -wave_max(-x); }

// The X^T / Y^T operand matrices (a few rows of f16, row stride ld, ld a multiple
// of 32) keep entry j of row n in 8-element chunk (j / 8) XOR (n & 3): the rows one
// fragment read touches then fall in different LDS banks.
__device__ __forceinline__ int xoff(int n, int j, int ld) { return n * ld + ((((j >> 3) ^ n) & 3) | ((j >> 3) & ~3)) * 8 + (j & 7); }

// Row n (< nx, else zero) of an operand matrix, entries j0 .. j0+7 (j0 % 8 == 0).
__device__ __forceinline__ f16x8_t xfrag(const _Float16* sx, int ld, int n, int nx, int j0) {
    if (n >= nx) return f16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
    return __builtin_bit_cast(f16x8_t, *(const u32x4_t*)(sx + xoff(n, j0, ld)));
}

// Key order inside one 32-key chunk of the FMA (slow) path. Lane (g, n)'s 8 K slots
// of a fragment hold keys j0 + 4 g + t (t < 4) and j0 + 16 + 4 g + (t - 4) (t >= 4).
// Everything indexed by key within a chunk (X^T fragments, the lane's keys) follows
// it; sums over K do not depend on the order.
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4_t pack_e(const float (&e)[8]) {
    return u32x4_t{pk_f16(e[0], e[1]), pk_f16(e[2], e[3]), pk_f16(e[4], e[5]), pk_f16(e[6], e[7])};
}

// -1 where the compiler cannot fold it: x - h for an f16 h is then one mixed-precision FMA that
// rounds to f16, where a subtraction converts h, subtracts and converts back.
__device__ __forceinline__ float minus_one() {
    float m = -1.f;
    asm("" : "+s"(m));
    return m;
}
// A packed f16 pair or fragment as it is stored: what is computed from it reads these bits (the
// compiler would otherwise round the floats again, an unrounded product among them).
template <typename V>
__device__ __forceinline__ V as_stored(V x) {
    asm("" : "+v"(x));
    return x;
}
// What pack_e's rounding leaves of each e, as f16.
__device__ __forceinline__ u32x4_t pack_e_lo(const float (&e)[8], const u32x4_t& hi, float m1) {
    const f16x8_t h = __builtin_bit_cast(f16x8_t, hi);
    f16x8_t l;
#pragma unroll
    for (int t = 0; t < 8; ++t) l[t] = (_Float16)fmaf((float)h[t], m1, e[t]);
    return __builtin_bit_cast(u32x4_t, l);
}

// e for one row (c, m) and the lane's 8 keys kv[0..7] (in the order above),
// exponent arguments by FMA.
__device__ __forceinline__ u32x4_t efrag(float c, float m, const float* kv) {
    float e[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) e[t] = __builtin_amdgcn_exp2f(fmaf(c, kv[t], m));
    return pack_e(e);
}

// Exponent arguments on the matrix cores: x = c k + m as a 32 (keys) x 32 (rows)
// product with K = 5 of 8 slots used, from f16 hi + lo parts of c, k and m:
//   keys (lane half g, key l % 32):   g = 0: (k_hi, k_hi, 1, 1)   g = 1: (k_lo, 0, 0, 0)
//   rows (lane half g, row l % 32):   (c_hi, c_lo, m_hi, m_lo) for both halves
// giving c_hi k_hi + c_lo k_hi + m_hi + m_lo + c_hi k_lo: every product is exact in
// the float accumulator and only c_lo k_lo (relative 2^-22 of c k) is left out.
__device__ __forceinline__ f16x4_t key_frag(float k, int g) {
    const _Float16 hi = (_Float16)k, lo = (_Float16)(k - (float)hi);
    if (g == 0) return f16x4_t{hi, hi, (_Float16)1.f, (_Float16)1.f};
    if (g == 1) return f16x4_t{lo, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
    return f16x4_t{(_Float16)0.f, (_Float16)0.f, (_Float16)0.f, (_Float16)0.f};
}

__device__ __forceinline__ f16x4_t row_rec(float c, float m) {
    const _Float16 ch = (_Float16)c, mh = (_Float16)m;
    return f16x4_t{ch, (_Float16)(c - (float)ch), mh, (_Float16)(m - (float)mh)};
}

// X^T fragment of row n (< nx, else zero) for the chunk at j0, keys in the order above.
__device__ __forceinline__ f16x8_t xfrag_perm(const _Float16* sx, int ld, int n, int nx, int j0, int g) {
    if (n >= nx) return f16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
    const f16x4_t lo = *(const f16x4_t*)(sx + xoff(n, j0 + 4 * g, ld));
    const f16x4_t hi = *(const f16x4_t*)(sx + xoff(n, j0 + 16 + 4 * g, ld));
    return f16x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
}

typedef float f32x16_t __attribute__((ext_vector_type(16)));

// The lane's 8 keys (order above) from the float key array.
__device__ __forceinline__ void keys_perm(const float* sk, int j0, int g, float (&kv)[8]) {
    *(u32x4_t*)kv = *(const u32x4_t*)(sk + j0 + 4 * g);
    *(u32x4_t*)(kv + 4) = *(const u32x4_t*)(sk + j0 + 16 + 4 * g);
}

// Exponent arguments go through the matrix cores when every c, m and k of the
// wave fits f16 with margin; otherwise (extreme logits) through FMAs. The forward
// and the backward take the same decision from the same values.
constexpr float ATT_F16_SAFE = 16384.f;

// Write quantity x / s as an f16 hi + lo pair into rows (row, row + 1) of X^T.
__device__ __forceinline__ void put_pair(_Float16* sx, int ld, int row, int j, float xs) {
    const _Float16 h = (_Float16)xs;
    sx[xoff(row, j, ld)] = h;
    sx[xoff(row + 1, j, ld)] = (_Float16)(xs - (float)h);
}

// Which block of row tiles a wave owns (direct sums).
struct WaveRows {
    int w;       // part of the sample (0 .. W-1)
    int t0, nt;  // first tile, tiles owned
};
template <int W>
__device__ __forceinline__ WaveRows wave_rows(int wave, int ntile) {
    WaveRows o;
    o.w = W == 1 ? 0 : wave;
    const int per = (((ntile + W - 1) / W) + 1) & ~1;  // even, <= ATT_NT for the W chosen at launch
    o.t0 = o.w * per;
    o.nt = ntile - o.t0 < per ? ntile - o.t0 : per;
    if (o.nt < 0) o.nt = 0;
    return o;
}

// Setup reads every per-sample operand a lane needs with one batch of loads
// (indices clamped to the valid range, so each load is issued; values past r are
// replaced by zeros), then works from registers.
//   keys / values: lane holds j = 64 u + lane, u < KPL (KPL * 64 >= rpad)
//   the wave's rows: lane holds il = 64 u + lane, u < RPL (RPL * 64 >= 16 NT)
template <int KPL>
__device__ __forceinline__ void load_keys(const float* pv, const float* pk, int r, int lane, float (&k)[KPL],
                                          float (&v)[KPL]) {
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        const int j = 64 * u + lane;
        const int jc = j < r ? j : r - 1;
        k[u] = pk[jc];
        v[u] = pv[jc];
    }
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        if (64 * u + lane >= r) k[u] = v[u] = 0.f;
    }
}

template <int NT>
struct RowsPerLane {
    static constexpr int value = (16 * NT + 63) / 64;
};

// rows t0 * 16 + il of quantity x (zero past r or past the rows in range)
template <int RPL>
__device__ __forceinline__ void load_rows(const float* x, int r, int t0, int nrows, int lane, float (&out)[RPL]) {
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
        const int il = 64 * u + lane, i = t0 * 16 + il;
        out[u] = x[i < r ? i : r - 1];
    }
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
        const int il = 64 * u + lane, i = t0 * 16 + il;
        if (!(il < nrows && i < r)) out[u] = 0.f;
    }
}

// key range over the keys held (valid keys only)
template <int KPL>
__device__ __forceinline__ void key_range(const float (&k)[KPL], int r, int lane, float& kmin, float& kmax) {
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        if (64 * u + lane < r) {
            lo = fminf(lo, k[u]);
            hi = fmaxf(hi, k[u]);
        }
    }
    kmin = wave_min(lo);
    kmax = wave_max(hi);
}

// (c_i, m_i) = (q_i log2(e) / tau, -c_i k*_i) of rows 64 u + lane (rows past r hold
// q = 0, so c = m = 0), and the largest |c|, |m| over rows below nrows together with
// the key range (wave-uniform). The exponent arguments go through the matrix cores
// when that maximum stays below ATT_F16_SAFE.
template <int RPL>
__device__ __forceinline__ float row_consts(const float (&q)[RPL], int lane, int nrows, float inv_tau, float kmin,
                                            float kmax, float (&c)[RPL], float (&m)[RPL]) {
    float big = fmaxf(fabsf(kmin), fabsf(kmax));
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
        c[u] = q[u] * (LOG2E * inv_tau);
        m[u] = -(c[u] * (c[u] >= 0.f ? kmax : kmin));
        if (64 * u + lane < nrows) big = fmaxf(big, fmaxf(fabsf(c[u]), fabsf(m[u])));
    }
    return wave_max(big);
}

// Largest of the W per-wave values in the sample's slots (each wave wrote slot[k] of
// its own area at stride `stride` floats; slot0 is the first wave's area).
template <int W>
__device__ __forceinline__ float sample_max(const float* slot0, int stride, int k) {
    float x = slot0[k];
#pragma unroll
    for (int w = 1; w < W; ++w) x = fmaxf(x, slot0[w * stride + k]);
    return x;
}

// X^T of the forward: f16 hi + lo pairs of quantities summed against e, row stride
// rpad. Quantity rows (the MFMA's M index): 0, 1: v / vs; 2: 1 for the real keys;
// 3: zero (not stored); 4, 5: v k / vks; 6, 7: k / ks. Output lanes 0-15 get
// (sum e v, sum e) for o and Z, lanes 16-31 the backward's row sums
// W1 = sum_j e v_j k_j and W2 = sum_j e k_j, from the same MFMAs.
constexpr int ATT_XROWS = 7;
__device__ __forceinline__ int xrow(int n) { return n < 3 ? n : n - 1; }
__device__ __forceinline__ f16x8_t xfrag_fwd(const _Float16* sx, int ld, int n, int j0, int g) {
    if (n == 3 || n > 7) return f16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
    return xfrag_perm(sx, ld, xrow(n), ATT_XROWS, j0, g);
}

// Exponent arguments of 32 keys x 32 rows from one v_mfma_f32_32x32x8_f16 (the key
// and row records of key_frag / row_rec use only 8 K slots): lane l gets row l % 32 and
// keys 8 a + 4 (l / 32) + t in element 4 a + t. Elements 8 p .. 8 p + 7 are the B
// operand of a 16x16x32 weighted sum over keys 16 p .. 16 p + 15 whose columns are
// rows n (lanes 0-15, 32-47) and n + 16 (lanes 16-31, 48-63): frag32 gives the
// quantities of row n to output slots 0-7 and those of row n + 16 to slots 8-15.
// X^T fragment for such a sum at keys jb .. jb + 15: lane (g4, q) with q % 8 a
// quantity row (row 3 and rows of the other half read as zero).
__device__ __forceinline__ f16x8_t frag32(const _Float16* sx, int ld, int lane, int jb) {
    const int qs = lane & 15, g4 = lane >> 4, q = qs & 7, h = g4 >> 1;
    if ((qs >> 3) != (g4 & 1) || q == 3) return f16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
    const int row = xrow(q);
    const f16x4_t lo = *(const f16x4_t*)(sx + xoff(row, jb + 4 * h, ld));
    const f16x4_t hi = *(const f16x4_t*)(sx + xoff(row, jb + 8 + 4 * h, ld));
    return f16x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
}

// ---------------------------------------------------------------------------
// Panel sums (the path almost every sample takes). The scores of one sample are a rank-one
// matrix: with the keys mapped to s_j = (k_j - kc) / Hk in [-1, 1] (kc, Hk: centre and half
// width of their range) and y_i = q_i log2(e) / tau * Hk, the exponent of row i and key j
// is y_i s_j - |y_i|. A row's sums are therefore values of functions of the one scalar y,
//   F_w(y) = sum_j w_j 2^(y s_j)      (w = 1, v; their derivatives give w s),
// and a key's sums values of functions of s. The range [-Y, Y] of y (of s: [-1, 1]) is cut
// into n panels of half width h <= rho (Y / n for s); inside the panel at y_p
//   2^(y s) = 2^(y_p s) e^(x s),   x = (y - y_p) ln 2,  |x s| <= rho ln 2,
// and e^t is a polynomial of degree 7 (relative error 5e-7 and its derivative's 5e-6 on the forward's
// panels, 2.5e-6 on the backward's wider ones). So one exponential per (panel, key) is enough:
// the moments sum_j w_j s_j^t 2^(y_p s_j - |y_p|), t = 0 .. 7, run on the matrix cores (A
// operand: the w s^t as f16 hi + lo pairs; B operand: the exponentials, 16 panels x 32 keys
// per v_mfma_f32_16x16x32_f16), and each row evaluates its panel's polynomials and their
// derivatives by Horner's rule in float. n = 16 ceil(Y / 24) (/ 32 in the backward, which
// needs no derivative) is 16 to 48 for the scores of a freshly drawn layer (|logits| up to
// 30 or so) and 128 (96 in the backward) when they reach 130, against r = 256 .. 1024
// exponentials per row for the direct sums; those stay for samples whose scores need more than
// 3 r / 8 (r / 4) panels or exceed the f16 range, and for small ranks.
// The backward's exponentials too are f16 hi + lo pairs. The direct sums round them once, but there
// a row's Z, o and column-sum terms share the rounded values, so that part of the error leaves with
// the division by Z. Panels of rows and panels of keys round different exponentials: with one f16
// each, o and D are as close to float64 as the direct ones (0.98 to 1.03 of their error), but the
// backward's sums 1.2 to 5 times further off (24 draws, rank 512, spread 9: gk 4.7e-4 against 1.9e-4, gv
// 4.8e-4 against 7.9e-5; rank 1024, spread 1: 5.8e-4 / 3.0e-4, 5.0e-4 / 2.5e-4). With pairs there what is
// left comes from the forward's Z and o, and is the direct form's error or less (1.3e-4, 4.6e-5; 9.2e-5,
// 3.4e-5). Pairs in the forward as well would leave 1e-5 (and cost it 9%).
// Measured (direct -> panel sums, us per launch alone, |logits| up to 30): batch 8192, rank
// 1024: forward 727 -> 88, backward 747 -> 119; batch 4096, rank 512: 106 -> 28, 108 -> 40;
// batch 4096, rank 256: 32 -> 15, 32 -> 19; with ten times the logits, rank 1024: 728 -> 381,
// 746 -> 496. (The backward's pairs cost 2 to 12% of that.) What remains is bound by
// the vector work around the exponentials (the tiles' powers, the polynomials) and the traffic of
// [v|q|k], h and the statistics. Where a line between the two forms lies: a panel costs what 2
// (forward) or 2.3 (backward) of a row's r direct exponentials cost (rank 256, batch 4096: 0.25 and
// 0.29 us against 0.126), on top of the set-up, and below ranks 128 and 192 the direct sums
// take no longer than the panels' set-up (rank 128, batch 8192: forward 23 -> 15; rank 64, panels
// forced: 12.5 -> 13.7, 13 -> 21). A sample beyond the line pays for the choice and for the
// panel kernels' registers: against kernels of the direct sums alone, |logits| of 500 and more,
// rank 1024 726 -> 756 and 746 -> 747, rank 512 112 -> 115 and 109 -> 114, rank 256 32.2 -> 35.5 and
// 32.4 -> 34 us.
//
// Data are handled in tiles of 128 entries, two consecutive entries per lane. A tile's
// operand matrix is kept in LDS as chunks of 8 entries x 16 rows (16 bytes per row and
// chunk, chunk pitch 272 bytes): the two-entry writes of a row fall in distinct banks
// and a fragment read takes 256 consecutive bytes per 16 lanes.
// ---------------------------------------------------------------------------
constexpr float AP_RHO_FWD = 1.5f, AP_RHO_BWD = 2.f;
constexpr int AP_MIN_RANK_FWD = 128, AP_MIN_RANK_BWD = 192;  // below them the direct sums are as fast
// groups of 16 panels per sweep over the entries
constexpr int AP_G_FWD = 6;
__host__ __device__ constexpr int ap_groups_bwd(int W) { return W == 1 ? 6 : 4; }
constexpr int AP_PITCH = 136;                 // f16 per chunk (16 rows x 8 entries + 8)
constexpr int AP_MAT = 16 * AP_PITCH;         // f16 of one operand matrix of a tile
constexpr float LN2 = 0.6931471805599453f;
// e^t by polynomials of degree 7, least squares in relative error: on |t| <= 1.5 ln 2 together with
// the derivative, and on |t| <= 2 ln 2
__device__ constexpr float AP_POLY_FWD[8] = {0.999999765f, 1.00000302f,   0.500008918f,  0.16664851f,
                                             0.0416248407f, 0.00835892749f, 0.00144744797f, 0.000191044982f};
__device__ constexpr float AP_POLY_BWD[8] = {0.999999162f, 1.00001286f,   0.500026441f,  0.166610319f,
                                             0.0415757685f, 0.00838847365f, 0.00147708824f, 0.000188074344f};

// Orders a wave's LDS accesses: what its lanes wrote before is what they read after.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
template <int W>
__device__ __forceinline__ void sample_sync() {
    if constexpr (W == 1) wave_sync();
    else __syncthreads();
}

// A workgroup holds four samples of one wave each, or one sample of W waves.
__host__ __device__ constexpr int att_block_waves(int W) { return W == 1 ? 4 : W; }
__host__ __device__ constexpr int att_block_samples(int W) { return W == 1 ? 4 : 1; }

// Panels of half width at most rho over [-Y, Y], in groups of 16.
struct Panels {
    int n;
    float h, inv2h;  // half width, and panels per unit of y
};
__device__ __forceinline__ Panels make_panels(float Y, float rho) {
    Panels p;
    const int g = (int)ceilf(Y * (1.f / (16.f * rho)));
    p.n = 16 * (g < 1 ? 1 : g);
    p.h = Y / (float)p.n;
    p.inv2h = Y > 1e-20f ? 0.5f * (float)p.n / Y : 0.f;
    return p;
}
__device__ __forceinline__ int panel_of(const Panels& p, float y, float Y) {
    const int i = (int)((y + Y) * p.inv2h);
    return i < 0 ? 0 : (i < p.n ? i : p.n - 1);
}

// Rows row .. row + 7 of a tile's hi and lo matrices: w z^t of entries 2 lane, 2 lane + 1.
__device__ __forceinline__ void put_powers(_Float16* hi, _Float16* lo, int row, int lane, float2 w, float2 z) {
    const int off = (lane >> 2) * AP_PITCH + ((2 * lane) & 7) + row * 8;
    const float m1 = minus_one();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        w = make_float2(as_stored(w.x), as_stored(w.y));  // the float product: the pair is its hi and lo part
        const uint32_t h = as_stored(pk_f16(w.x, w.y));
        const f16x2_t hv = __builtin_bit_cast(f16x2_t, h);
        const f16x2_t lv = {(_Float16)fmaf((float)hv.x, m1, w.x), (_Float16)fmaf((float)hv.y, m1, w.y)};
        *(uint32_t*)(hi + off + 8 * t) = h;
        *(uint32_t*)(lo + off + 8 * t) = __builtin_bit_cast(uint32_t, lv);
        w.x *= z.x;
        w.y *= z.y;
    }
}
// A operand of entries 32 ks .. + 31: lane l has row l % 16, entries 8 (l / 16) .. + 7.
__device__ __forceinline__ f16x8_t panel_frag(const _Float16* x, int ks, int lane) {
    return __builtin_bit_cast(f16x8_t, *(const u32x4_t*)(x + (4 * ks + (lane >> 4)) * AP_PITCH + (lane & 15) * 8));
}

// p(x) and p'(x) of a polynomial of degree 7.
__device__ __forceinline__ void horner_d(const float* c, float x, float& p, float& d) {
    p = c[7];
    d = 0.f;
#pragma unroll
    for (int t = 6; t >= 0; --t) {
        d = fmaf(d, x, p);
        p = fmaf(p, x, c[t]);
    }
}
__device__ __forceinline__ float horner(const float* c, float x) {
    float p = c[7];
#pragma unroll
    for (int t = 6; t >= 0; --t) p = fmaf(p, x, c[t]);
    return p;
}

// A copy the compiler knows nothing about: what is computed from it inside a loop stays
// there (hoisted out of the sweep loop, the tiles' powers alone would fill the registers).
__device__ __forceinline__ float2 in_loop(float2 x) {
    asm volatile("" : "+v"(x.x), "+v"(x.y));
    return x;
}

// Two consecutive values of a row of length r (zeros past it; r is a multiple of 8).
__device__ __forceinline__ float2 load_pair(const float* x, int j, int r) {
    return *(const float2*)(x + (j < r ? j : r - 2));
}
__device__ __forceinline__ float2 pair_or_zero(float2 x, bool ok) {
    return make_float2(ok ? x.x : 0.f, ok ? x.y : 0.f);
}
__device__ __forceinline__ float abs_max2(float m, float2 x) { return fmaxf(m, fmaxf(fabsf(x.x), fabsf(x.y))); }

// Maxima over a sample of per-wave values held in x[0 .. N - 1] (every lane gets them).
template <int W, int N>
__device__ __forceinline__ void sample_maxima(float* slots, int wave, int lane, float (&x)[N]) {
#pragma unroll
    for (int e = 0; e < N; ++e) x[e] = wave_max(x[e]);
    if constexpr (W > 1) {
        if (lane == 0) {
#pragma unroll
            for (int e = 0; e < N; ++e) slots[wave * N + e] = x[e];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < N; ++e)
#pragma unroll
            for (int w = 0; w < W; ++w) x[e] = fmaxf(x[e], slots[w * N + e]);
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < N; ++e) x[e] = uniform_f(x[e]);
}

// Scores of one sample as the panel sums see them.
struct ScoreRange {
    float kc, Hk, iHk, Y;  // key centre and half width (and 1 / Hk), largest |y|
    Panels p;
    bool panels;           // panel sums, else direct sums
};
// kneg = -min k, kmax and qmax = max |q| over the sample; most: the most panels worth having.
__device__ __forceinline__ ScoreRange score_range(float kneg, float kmax, float qmax, float inv_tau, int most, float rho) {
    ScoreRange o;
    o.kc = 0.5f * (kmax - kneg);
    o.Hk = 0.5f * (kmax + kneg);
    o.iHk = o.Hk > 1e-30f ? 1.f / o.Hk : 0.f;
    const float cmax = qmax * (LOG2E * inv_tau), ka = fmaxf(fabsf(kneg), fabsf(kmax));
    o.Y = cmax * o.Hk;
    const bool safe = fmaxf(fmaxf(ka, cmax), cmax * ka) < ATT_F16_SAFE;  // then Y is below 2 ATT_F16_SAFE
    o.p = make_panels(safe ? o.Y : 0.f, rho);
    o.panels = safe && o.p.n <= most;
    return o;
}

// LDS of the forward's panel sums, in floats: per wave a tile's hi and lo matrices and its
// s values, reused for the wave's moments and the panels' polynomials (pitch 20: rows at
// random panels fall in all banks). With one wave per sample the polynomials take the
// place of the tile; four waves keep group g's behind the moments of wave g % 4.
constexpr int AP_FWD_WAVE = AP_MAT + 128;
constexpr int AP_FWD_PITCH = 20;
static_assert(16 * AP_G_FWD * AP_FWD_PITCH <= AP_FWD_WAVE, "the polynomials fit the tile");
static_assert(256 * AP_G_FWD + 16 * AP_FWD_PITCH * ((AP_G_FWD + 3) / 4) <= AP_FWD_WAVE,
              "a wave's moments and a quarter of the polynomials fit the tile");

// Direct sums (the samples the panel sums leave): LDS per sample (shared by its W waves):
// keys, X^T. Per wave: row constants and one slot for the range check.
__host__ __device__ constexpr int attn_fwd_sample_floats(int rpad) { return rpad + ATT_XROWS * rpad / 2; }
__host__ __device__ constexpr int attn_fwd_wave_floats() { return 2 * 16 * ATT_NT + 4; }
// (with one wave per sample they lie inside the wave's panel area)
__host__ __device__ constexpr int attn_fwd_direct_floats(int rpad, int W) {
    return attn_fwd_sample_floats(rpad) + W * attn_fwd_wave_floats();
}
static_assert(attn_fwd_direct_floats(16 * ATT_NT, 1) <= AP_FWD_WAVE, "one sample's direct sums fit its wave's area");
__host__ __device__ constexpr int attn_fwd_panel_floats(int W) {
    return att_block_waves(W) * AP_FWD_WAVE + (W > 1 ? 4 * W : 0);
}
__host__ __device__ constexpr int attn_fwd_block_floats(int rpad, int W) {
    return W > 1 && attn_fwd_direct_floats(rpad, W) > attn_fwd_panel_floats(W) ? attn_fwd_direct_floats(rpad, W)
                                                                               : attn_fwd_panel_floats(W);
}

// What the forward writes of row i. stats: [o | Z | D] per sample, row stride 3 r.
template <typename T>
struct FwdOut {
    T* H;
    void* H2;
    bool h2_f16;
    float* so;
    int r;
    int* err;
};

// Panel sums of one sample. k, v, q: the wave's tiles w, w + W, ... (zeros past r).
template <typename T, int W, int TPW>
__device__ __forceinline__ void attn_fwd_panels(const ScoreRange& R, int r, float alpha, float beta, float inv_tau,
                                                const float2 (&k)[TPW], const float2 (&v)[TPW], const float2 (&q)[TPW],
                                                float vmax, float* smem, int wave, int w, int lane,
                                                const FwdOut<T>& out) {
    constexpr int AP_G = AP_G_FWD;
    float* const region = smem + wave * AP_FWD_WAVE;
    _Float16* const xh = (_Float16*)region;
    _Float16* const xl = xh + AP_MAT;
    float* const ts = region + AP_MAT;
    auto coef = [&](int p) {  // polynomials of panel p of the sweep
        return W == 1 ? region + p * AP_FWD_PITCH
                      : smem + ((p >> 4) & 3) * AP_FWD_WAVE + 256 * AP_G + ((p >> 6) * 16 + (p & 15)) * AP_FWD_PITCH;
    };
    const float vs = pow2_ceil(vmax), ivs = 1.0f / vs;  // exact scaling: a power of two
    const float cq = LOG2E * inv_tau * R.Hk;
    const int ng = R.p.n / 16, col = lane & 15;
    float2 ov[TPW], zv[TPW], dv[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) ov[i] = zv[i] = dv[i] = make_float2(0.f, 0.f);
    for (int g0 = 0; g0 < ng; g0 += AP_G) {
        const int gc = ng - g0 < AP_G ? ng - g0 : AP_G;
        f32x4_t acc[AP_G];
        float yp[AP_G];
#pragma unroll
        for (int g = 0; g < AP_G; ++g) {
            acc[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            yp[g] = fmaf((float)(2 * (16 * (g0 + g) + col) + 1), R.p.h, -R.Y);
        }
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int j0 = 128 * (w + W * i);
            if (j0 < r) {
                const bool ok = j0 + 2 * lane < r;
                const float2 kk = in_loop(k[i]), vv = in_loop(v[i]);
                const float2 s = pair_or_zero(make_float2((kk.x - R.kc) * R.iHk, (kk.y - R.kc) * R.iHk), ok);
                wave_sync();
                put_powers(xh, xl, 0, lane, ok ? make_float2(1.f, 1.f) : make_float2(0.f, 0.f), s);
                put_powers(xh, xl, 8, lane, make_float2(vv.x * ivs, vv.y * ivs), s);
                *(float2*)(ts + 2 * lane) = s;
                wave_sync();
                const int nks = r - j0 < 128 ? (r - j0 + 31) / 32 : 4;
#pragma unroll 1
                for (int ks = 0; ks < nks; ++ks) {
                    const f16x8_t ah = panel_frag(xh, ks, lane), al = panel_frag(xl, ks, lane);
                    float s8[8];
                    *(f32x4_t*)s8 = *(const f32x4_t*)(ts + 32 * ks + 8 * (lane >> 4));
                    *(f32x4_t*)(s8 + 4) = *(const f32x4_t*)(ts + 32 * ks + 8 * (lane >> 4) + 4);
#pragma unroll
                    for (int g = 0; g < AP_G; ++g)
                        if (g < gc) {
                            float e[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) e[u] = __builtin_amdgcn_exp2f(fmaf(yp[g], s8[u], -fabsf(yp[g])));
                            const f16x8_t ef = __builtin_bit_cast(f16x8_t, pack_e(e));
                            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, ef, acc[g], 0, 0, 0);
                            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, ef, acc[g], 0, 0, 0);
                        }
                }
            }
        }
        // lane (q4, col) holds moments 4 (q4 % 2) .. + 3 of the 1 (q4 < 2) and v sums of panel col
        wave_sync();
        const bool odd = (lane >> 4) & 1;
        const float sc = lane >= 32 ? vs : 1.f;
        if constexpr (W == 1) {
#pragma unroll
            for (int g = 0; g < AP_G; ++g)
                if (g < gc) {
                    f32x4_t x = acc[g];
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[e] *= sc * (odd ? AP_POLY_FWD[4 + e] : AP_POLY_FWD[e]);
                    *(f32x4_t*)(coef(16 * g + col) + 4 * (lane >> 4)) = x;
                }
        } else {
#pragma unroll
            for (int g = 0; g < AP_G; ++g)
                if (g < gc) *(f32x4_t*)(region + (g * 64 + lane) * 4) = acc[g];
            __syncthreads();
            for (int g = w; g < gc; g += W) {  // the waves' parts, in wave order
                f32x4_t x = *(const f32x4_t*)(smem + (g * 64 + lane) * 4);
#pragma unroll
                for (int p = 1; p < W; ++p) x += *(const f32x4_t*)(smem + p * AP_FWD_WAVE + (g * 64 + lane) * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] *= sc * (odd ? AP_POLY_FWD[4 + e] : AP_POLY_FWD[e]);
                *(f32x4_t*)(coef(16 * g + col) + 4 * (lane >> 4)) = x;
            }
        }
        sample_sync<W>();
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            if (128 * (w + W * i) >= r) continue;
            const float2 qi = in_loop(q[i]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float y = (e ? qi.y : qi.x) * cq;
                const int p = panel_of(R.p, y, R.Y), pl = p - 16 * g0;
                const bool mine = pl >= 0 && pl < 16 * gc;
                const float ypi = fmaf((float)(2 * p + 1), R.p.h, -R.Y), x = (y - ypi) * LN2;
                const float* const cp = coef(mine ? pl : 0);
                float c[16];
#pragma unroll
                for (int u = 0; u < 4; ++u) *(f32x4_t*)(c + 4 * u) = *(const f32x4_t*)(cp + 4 * u);
                float z, zs, sv, ss;
                horner_d(c, x, z, zs);
                horner_d(c + 8, x, sv, ss);
                const float rz = __builtin_amdgcn_rcpf(z), o = sv * rz;
                const float D = (ss - o * zs) * rz * R.Hk;
                const float zi = z * __builtin_amdgcn_exp2f(fabsf(ypi) - fabsf(y));
                if (mine) {
                    if (e) { ov[i].y = o; zv[i].y = zi; dv[i].y = D; }
                    else { ov[i].x = o; zv[i].x = zi; dv[i].x = D; }
                }
            }
        }
        // the next sweep's tiles overwrite polynomials that other waves of the sample still read
        if (W > 1 && g0 + AP_G < ng) __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int j = 128 * (w + W * i) + 2 * lane;
        if (j >= r) continue;
        const float h0 = beta * v[i].x + alpha * ov[i].x, h1 = beta * v[i].y + alpha * ov[i].y;
        *(uint32_t*)(out.H + j) = pack_bf16x2(h0, h1);
        if (out.H2 && out.h2_f16) {  // h as f16, the up projection's operand
            *(uint32_t*)((_Float16*)out.H2 + j) = pk_f16(h0, h1);
            if (fmaxf(fabsf(h0), fabsf(h1)) >= F16_OVERFLOW) atomicOr(out.err, 2);  // f16 range bit of the error word
        } else if (out.H2) {         // lo part of a hi + lo pair
            *(uint32_t*)((T*)out.H2 + j) = pack_bf16x2(h0 - st<T>::round(h0), h1 - st<T>::round(h1));
        }
        *(float2*)(out.so + j) = ov[i];
        *(float2*)(out.so + r + j) = zv[i];
        *(float2*)(out.so + 2 * r + j) = dv[i];
    }
}

// Direct sums of one sample. NT: tiles computed per wave (a power of two >= the tiles it
// owns; the extra ones are computed on harmless row constants and discarded). KB: 256-key
// batches a lane's registers cover (4 KB >= rpad / 64).
template <typename T, int W, int NT, int KB>
__device__ __forceinline__ void attn_fwd_direct(int r, int rpad, float alpha, float beta, float inv_tau,
                                                const float* __restrict__ pv, float* sk, int lane, int wave,
                                                const FwdOut<T>& out) {
    // sk: [rpad] keys (shared by the sample's waves)
    const WaveRows wr = wave_rows<W>(wave, rpad / 16);
    _Float16* sx = (_Float16*)(sk + rpad);                   // X^T (ATT_XROWS stored rows)
    float* pw = sk + attn_fwd_sample_floats(rpad);
    float2* scm = (float2*)(pw + wr.w * attn_fwd_wave_floats());   // [16 ATT_NT] row constants
    float* slot = pw + wr.w * attn_fwd_wave_floats() + 2 * 16 * ATT_NT;
    constexpr int KPL = 4 * KB;
    constexpr int RPL = RowsPerLane<NT>::value;
    float kr[KPL], vr[KPL], qr[RPL];
    load_keys<KPL>(pv, pv + 2 * r, r, lane, kr, vr);
    load_rows<RPL>(pv + r, r, wr.t0, 16 * NT, lane, qr);
    float kmin, kmax;
    key_range<KPL>(kr, r, lane, kmin, kmax);
    float vmax = 0.f, mvk = 0.f, mk = 0.f;
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        vmax = fmaxf(vmax, fabsf(vr[u]));
        mvk = fmaxf(mvk, fabsf(vr[u] * kr[u]));
        mk = fmaxf(mk, fabsf(kr[u]));
    }
    // exact scalings: powers of two, identical in every wave of the sample (all see all keys)
    const float vs = uniform_f(pow2_ceil(wave_max(vmax))), ivs = 1.0f / vs;
    const float vks = uniform_f(pow2_ceil(wave_max(mvk))), ivks = 1.0f / vks;
    const float ks = uniform_f(pow2_ceil(wave_max(mk))), iks = 1.0f / ks;
    const int ldx = rpad;
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        const int j = 64 * u + lane;
        if (j < rpad && u % W == wr.w) {
            sk[j] = kr[u];
            put_pair(sx, ldx, 0, j, vr[u] * ivs);
            sx[xoff(2, j, ldx)] = (_Float16)(j < r ? 1.f : 0.f);
            put_pair(sx, ldx, xrow(4), j, vr[u] * kr[u] * ivks);
            put_pair(sx, ldx, xrow(6), j, kr[u] * iks);
        }
    }
    float c[RPL], m[RPL];
    float big = row_consts<RPL>(qr, lane, 16 * wr.nt, inv_tau, kmin, kmax, c, m);
    if (W > 1) {  // one decision per sample, as in the backward
        if (lane == 0) slot[0] = big;
        __syncthreads();
        big = uniform_f(sample_max<W>(pw + 2 * 16 * ATT_NT, attn_fwd_wave_floats(), 0));
    }
    const bool fast = big < ATT_F16_SAFE;  // (infinities take the FMAs; the maxima pass over NaN, which spreads by itself)
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
        const int il = 64 * u + lane;
        if (il < 16 * NT) {
            if (fast) *(f16x4_t*)(scm + il) = row_rec(c[u], m[u]);
            else scm[il] = make_float2(c[u], m[u]);
        }
    }
    sample_sync<W>();
    const int g = lane >> 4, n = lane & 15;
    f32x4_t acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto chunks = [&](auto fast_c) {
        constexpr bool FAST = decltype(fast_c)::value;
        for (int j0 = 0; j0 < rpad; j0 += 32) {
            if (FAST) {
                // 32-row tiles: acc[tt] holds rows 32 tt + n (lanes 0-31) and 32 tt + 16 + n
                const f16x4_t kf = key_frag(sk[j0 + (lane & 31)], lane >> 5);
                const f16x8_t a0 = frag32(sx, ldx, lane, j0), a1 = frag32(sx, ldx, lane, j0 + 16);
                const f32x16_t z16 = {};
                // the next tile's arguments are issued before this tile's exponentials, so
                // the matrix core computes them while the wave's exponentials run
                f32x16_t xn = __builtin_amdgcn_mfma_f32_32x32x8f16(kf, *(const f16x4_t*)(scm + (lane & 31)), z16, 0, 0, 0);
#pragma unroll
                for (int tt = 0; tt < NT / 2; ++tt) {
                    const f32x16_t x = xn;
                    if (tt + 1 < NT / 2) {
                        const f16x4_t rec = *(const f16x4_t*)(scm + 32 * (tt + 1) + (lane & 31));
                        xn = __builtin_amdgcn_mfma_f32_32x32x8f16(kf, rec, z16, 0, 0, 0);
                    }
                    float e0[8], e1[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        e0[u] = __builtin_amdgcn_exp2f(x[u]);
                        e1[u] = __builtin_amdgcn_exp2f(x[8 + u]);
                    }
                    acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, __builtin_bit_cast(f16x8_t, pack_e(e0)), acc[tt], 0, 0, 0);
                    acc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, __builtin_bit_cast(f16x8_t, pack_e(e1)), acc[tt], 0, 0, 0);
                }
            } else {
                float kv[8];
                keys_perm(sk, j0, g, kv);
                const f16x8_t a = xfrag_fwd(sx, ldx, n, j0, g);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const float2 cm = scm[16 * t + n];
                    const u32x4_t e = efrag(cm.x, cm.y, kv);
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, __builtin_bit_cast(f16x8_t, e), acc[t], 0, 0, 0);
                }
            }
        }
    };
    if (fast) chunks(std::true_type{});
    else chunks(std::false_type{});
    // Which row and quantities each lane's accumulators hold. Fast path: 32-row tiles,
    // lane (g4, n) has quantities 4 (g4 & 1) .. +3 of row 16 (2 t + g4 / 2) + n. Slow
    // path: 16-row tiles, lanes 0-31 only, quantities 4 (lane / 16) .. +3 of row 16 t + n.
    const int na = fast ? NT / 2 : NT;
    const bool lo = fast ? ((lane >> 4) & 1) == 0 : lane < 16;
    // lo lanes: (sum e v, sum e) of their row; the lanes 16 above: (W1, W2), fetched from there
    float vi[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {  // all loads first
        const int t16 = fast ? 2 * t + (lane >> 5) : t;
        const int i = (wr.t0 + t16) * 16 + n;
        vi[t] = pv[i < r ? i : r - 1];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float w1 = __shfl_xor((acc[t].x + acc[t].y) * vks, 16), w2 = __shfl_xor((acc[t].z + acc[t].w) * ks, 16);
        const int t16 = fast ? 2 * t + (lane >> 5) : t;
        const int i = (wr.t0 + t16) * 16 + n;
        if (lo && t < na && t16 < wr.nt && i < r) {
            const float z = acc[t].z, rz = __builtin_amdgcn_rcpf(z);
            const float o = (acc[t].x + acc[t].y) * vs * rz;
            const float hv = beta * vi[t] + alpha * o;
            st<T>::store(out.H + i, hv);
            if (out.H2 && out.h2_f16) {  // h as f16, the up projection's operand
                ((_Float16*)out.H2)[i] = (_Float16)hv;
                if (fabsf(hv) >= F16_OVERFLOW) atomicOr(out.err, 2);  // f16 range bit of the error word
            } else if (out.H2) {         // lo part of a hi + lo pair
                st<T>::store((T*)out.H2 + i, hv - st<T>::round(hv));
            }
            out.so[i] = o;
            out.so[r + i] = z;
            out.so[2 * r + i] = (w1 - o * w2) * rz;
        }
    }
}

// stats: [o | Z | D] per sample, row stride 3 r. PANEL: samples choose between the two forms
// (smaller ranks take the direct sums).
template <typename T, int W, int NT, int KB, bool PANEL>
__global__ __launch_bounds__(64 * att_block_waves(W)) __attribute__((amdgpu_waves_per_eu(KB == 4 ? 3 : 4, 8))) void k_attn_fwd_mfma(
    int64_t B, int r, int rpad, float alpha, float beta, float inv_tau, const float* __restrict__ P, int64_t ldp,
    T* __restrict__ H, void* __restrict__ H2, int64_t ldh, bool h2_f16, float* __restrict__ stats, int* err) {
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int w = W == 1 ? 0 : wave;
    const int64_t b = (int64_t)blockIdx.x * att_block_samples(W) + (W == 1 ? wave : 0);
    if (b >= B) return;  // (one wave per sample only: with W > 1 there are B workgroups)
    const float* pv = P + b * ldp;
    const FwdOut<T> out{H + b * ldh, H2 ? (void*)((T*)H2 + b * ldh) : nullptr, h2_f16, stats + b * 3 * (int64_t)r, r, err};
    if constexpr (!PANEL) {
        attn_fwd_direct<T, W, NT, KB>(r, rpad, alpha, beta, inv_tau, pv, smem + wave * attn_fwd_direct_floats(rpad, 1), lane,
                                      wave, out);
        return;
    }
    constexpr int TPW = 2 * KB / W;  // 128-entry tiles of the wave
    float2 k[TPW], v[TPW], q[TPW];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int j = 128 * (w + W * i) + 2 * lane;
        v[i] = load_pair(pv, j, r);
        q[i] = load_pair(pv + r, j, r);
        k[i] = load_pair(pv + 2 * r, j, r);
    }
    float mx[4] = {-INFINITY, -INFINITY, 0.f, 0.f};  // -min k, max k, max |q|, max |v|
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const bool ok = 128 * (w + W * i) + 2 * lane < r;
        if (ok) {
            mx[0] = fmaxf(mx[0], fmaxf(-k[i].x, -k[i].y));
            mx[1] = fmaxf(mx[1], fmaxf(k[i].x, k[i].y));
        }
        v[i] = pair_or_zero(v[i], ok);
        q[i] = pair_or_zero(q[i], ok);
        mx[2] = abs_max2(mx[2], q[i]);
        mx[3] = abs_max2(mx[3], v[i]);
    }
    sample_maxima<W>(smem + attn_fwd_panel_floats(W) - 4 * W, wave, lane, mx);
    const ScoreRange R = score_range(mx[0], mx[1], mx[2], inv_tau, 3 * r / 8, AP_RHO_FWD);
    if (R.panels) attn_fwd_panels<T, W, TPW>(R, r, alpha, beta, inv_tau, k, v, q, mx[3], smem, wave, w, lane, out);
    else attn_fwd_direct<T, W, NT, KB>(r, rpad, alpha, beta, inv_tau, pv, W == 1 ? smem + wave * AP_FWD_WAVE : smem, lane, wave, out);
}

// LDS of the backward's panel sums, in floats: per wave three tile matrices (a z^t and
// a o z^t: hi, lo; go/Z z^t: hi in rows 0-7, lo in rows 8-15), reused for the wave's moments and the
// panels' polynomials (pitch 28) as in the forward. The tile's y values lie in the chunks' padding
// (entries 0-3 of a chunk behind its hi rows, 4-7 behind its lo rows): four waves then take 52 KB and
// three workgroups share a CU, the three waves per SIMD that the registers allow; with 512 bytes per
// wave of their own it was two (batch 8192, rank 1024: 147 -> 119 us, rank 512, batch 4096: 48 -> 40;
// samples left to the direct sums 780 -> 747 and 126 -> 114).
constexpr int AP_BWD_WAVE = 3 * AP_MAT / 2;
constexpr int AP_BWD_PITCH = 28;
static_assert(16 * ap_groups_bwd(1) * AP_BWD_PITCH <= AP_BWD_WAVE, "the polynomials fit the tile");
static_assert(512 * ap_groups_bwd(4) + 16 * AP_BWD_PITCH * ((ap_groups_bwd(4) + 3) / 4) <= AP_BWD_WAVE,
              "a wave's moments and a quarter of the polynomials fit the tile");

// Direct sums: LDS per sample (shared by its W waves): keys, row constants (8 bytes per
// row), Y^T (6 rows of f16 and two rows of zeros, row stride rpad); per wave four slots for
// the range check and the three scales.
__host__ __device__ constexpr int attn_bwd_sample_floats(int rpad) { return rpad + 2 * rpad + 4 * rpad; }
__host__ __device__ constexpr int attn_bwd_wave_floats() { return 4; }
__host__ __device__ constexpr int attn_bwd_direct_floats(int rpad, int W) {
    return attn_bwd_sample_floats(rpad) + W * attn_bwd_wave_floats();
}
static_assert(attn_bwd_direct_floats(16 * ATT_NT, 1) <= AP_BWD_WAVE, "one sample's direct sums fit its wave's area");
__host__ __device__ constexpr int attn_bwd_panel_floats(int W) {
    return att_block_waves(W) * AP_BWD_WAVE + (W > 1 ? 8 * W : 0);
}
__host__ __device__ constexpr int attn_bwd_block_floats(int rpad, int W) {
    return W > 1 && attn_bwd_direct_floats(rpad, W) > attn_bwd_panel_floats(W) ? attn_bwd_direct_floats(rpad, W)
                                                                               : attn_bwd_panel_floats(W);
}

// The backward's Y^T fragment, laid out as frag32's with K over rows and the 6
// quantity rows stored as they are. Every lane loads: the lanes whose slots hold no
// quantity (the other half's, and quantities 6 and 7) read row 7, which holds zeros,
// so the fragment needs no per-lane branches.
__device__ __forceinline__ f16x8_t yfrag32(const _Float16* sy, int ld, int lane, int jb) {
    const int qs = lane & 15, g4 = lane >> 4, q = qs & 7, h = g4 >> 1;
    const int row = ((qs >> 3) != (g4 & 1) || q >= 6) ? 7 : q;
    const f16x4_t lo = *(const f16x4_t*)(sy + xoff(row, jb + 4 * h, ld));
    const f16x4_t hi = *(const f16x4_t*)(sy + xoff(row, jb + 8 + 4 * h, ld));
    return f16x8_t{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
}

// Backward. With the forward's D_i = sum_j A_ij (v_j - o_i) k_j, dq_i = go_i / tau D_i needs no
// exponentials (go = alpha gh). The column sums C1_j = sum_i e_ij a_i, C2_j = sum_i e_ij a_i o_i,
// C3_j = sum_i e_ij go_i / Z_i (a_i = go_i q_i / (Z_i tau)) give dk_j = v_j C1_j - C2_j and
// dv_j = beta gh_j + C3_j. Panel sums: e_ij = 2^(y_i s_j - |y_i|) as a function of s_j, in panels
// of half width 1 / n at s_p; with z_i = y_i / Y, 2^(y_i (s - s_p)) = e^(x z_i) for
// x = Y (s - s_p) ln 2, so the moments are sum_i w_i z_i^t 2^(y_i s_p - |y_i|) over the rows.
// tk, tv, tg: the wave's tiles of k, v, gh; y, a, ao, gz: y_i, a_i, a_i o_i, go_i / Z_i (zeros past r).
template <typename T, int W, int TPW>
__device__ __forceinline__ void attn_bwd_panels(const ScoreRange& R, int r, float beta, const float2 (&tk)[TPW],
                                                const float2 (&tv)[TPW], const float2 (&tg)[TPW],
                                                const float2 (&y)[TPW], const float2 (&a)[TPW],
                                                const float2 (&ao)[TPW], const float2 (&gz)[TPW], float ma, float mb,
                                                float mc, float* smem, int wave, int w, int lane, T* gp) {
    float* const region = smem + wave * AP_BWD_WAVE;
    _Float16* const xh = (_Float16*)region;
    _Float16* const xl = xh + AP_MAT;
    _Float16* const xg = xl + AP_MAT;
    const int yw = (lane >> 2) * AP_PITCH + 128 + ((2 * lane) & 2) * 2;  // where the lane's two y go (f16 units)
    constexpr int AP_G = ap_groups_bwd(W);
    auto coef = [&](int p) {  // polynomials of panel p of the sweep
        return W == 1 ? region + p * AP_BWD_PITCH
                      : smem + ((p >> 4) & 3) * AP_BWD_WAVE + 512 * AP_G + ((p >> 6) * 16 + (p & 15)) * AP_BWD_PITCH;
    };
    const float as = pow2_ceil(ma), bs = pow2_ceil(mb), cs = pow2_ceil(mc);
    const float ias = 1.0f / as, ibs = 1.0f / bs, ics = 1.0f / cs;  // exact: powers of two
    const float iY = R.Y > 1e-20f ? 1.f / R.Y : 0.f, xs = R.Y * LN2;
    const int n = R.p.n, ng = n / 16, col = lane & 15;
    const float sh = 1.f / (float)n;  // half width of a panel of s
    const float m1 = minus_one();
    float2 c1[TPW], c3[TPW];  // dk, dv of the wave's keys
#pragma unroll
    for (int i = 0; i < TPW; ++i) c1[i] = c3[i] = make_float2(0.f, 0.f);
    for (int g0 = 0; g0 < ng; g0 += AP_G) {
        const int gc = ng - g0 < AP_G ? ng - g0 : AP_G;
        f32x4_t acc[AP_G], acg[AP_G];
        float sp[AP_G];
#pragma unroll
        for (int g = 0; g < AP_G; ++g) {
            acc[g] = acg[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            sp[g] = fmaf((float)(2 * (16 * (g0 + g) + col) + 1), sh, -1.f);
        }
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int j0 = 128 * (w + W * i);
            if (j0 < r) {
                const float2 yy = in_loop(y[i]), z = make_float2(yy.x * iY, yy.y * iY);
                const float2 wa = in_loop(a[i]), wo = in_loop(ao[i]), wg = in_loop(gz[i]);
                wave_sync();
                put_powers(xh, xl, 0, lane, make_float2(wa.x * ias, wa.y * ias), z);
                put_powers(xh, xl, 8, lane, make_float2(wo.x * ibs, wo.y * ibs), z);
                put_powers(xg, xg + 64, 0, lane, make_float2(wg.x * ics, wg.y * ics), z);
                *(float2*)(((lane & 2) ? xl : xh) + yw) = yy;
                wave_sync();
                const int nks = r - j0 < 128 ? (r - j0 + 31) / 32 : 4;
#pragma unroll 1
                for (int ks = 0; ks < nks; ++ks) {
                    const f16x8_t ah = panel_frag(xh, ks, lane), al = panel_frag(xl, ks, lane), ag = panel_frag(xg, ks, lane);
                    float y8[8];
                    *(f32x4_t*)y8 = *(const f32x4_t*)(xh + (4 * ks + (lane >> 4)) * AP_PITCH + 128);
                    *(f32x4_t*)(y8 + 4) = *(const f32x4_t*)(xl + (4 * ks + (lane >> 4)) * AP_PITCH + 128);
#pragma unroll
                    for (int g = 0; g < AP_G; ++g)
                        if (g < gc) {
                            float e[8];
#pragma unroll
                            for (int u = 0; u < 8; ++u) e[u] = __builtin_amdgcn_exp2f(fmaf(sp[g], y8[u], -fabsf(y8[u])));
                            const u32x4_t ep = as_stored(pack_e(e));
                            const f16x8_t ef = __builtin_bit_cast(f16x8_t, ep),
                                          el = __builtin_bit_cast(f16x8_t, pack_e_lo(e, ep, m1));
                            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, ef, acc[g], 0, 0, 0);
                            acg[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ag, ef, acg[g], 0, 0, 0);
                            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(al, ef, acc[g], 0, 0, 0);
                            acg[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ag, el, acg[g], 0, 0, 0);
                            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ah, el, acc[g], 0, 0, 0);
                        }
                }
            }
        }
        // lane (q4, col): acc moments 4 (q4 % 2) .. + 3 of the a (q4 < 2) and a o sums of panel col;
        // acg those of the go/Z sums, hi parts for q4 < 2, lo parts for the others
        wave_sync();
        const bool odd = (lane >> 4) & 1;
        const float sc = lane < 32 ? as : bs;
#pragma unroll
        for (int g = 0; g < AP_G; ++g)
            if (g < gc) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acg[g][e] += __shfl_xor(acg[g][e], 32);
            }
        auto put = [&](int g, f32x4_t x, f32x4_t xg4) {
            float* const c = coef(16 * g + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] *= sc * (odd ? AP_POLY_BWD[4 + e] : AP_POLY_BWD[e]);
                xg4[e] *= cs * (odd ? AP_POLY_BWD[4 + e] : AP_POLY_BWD[e]);
            }
            *(f32x4_t*)(c + 4 * (lane >> 4)) = x;
            if (lane < 32) *(f32x4_t*)(c + 16 + 4 * (lane >> 4)) = xg4;
        };
        if constexpr (W == 1) {
#pragma unroll
            for (int g = 0; g < AP_G; ++g)
                if (g < gc) put(g, acc[g], acg[g]);
        } else {
#pragma unroll
            for (int g = 0; g < AP_G; ++g)
                if (g < gc) {
                    *(f32x4_t*)(region + (g * 128 + lane) * 4) = acc[g];
                    *(f32x4_t*)(region + (g * 128 + 64 + lane) * 4) = acg[g];
                }
            __syncthreads();
            for (int g = w; g < gc; g += W) {  // the waves' parts, in wave order
                f32x4_t x = *(const f32x4_t*)(smem + (g * 128 + lane) * 4);
                f32x4_t xg4 = *(const f32x4_t*)(smem + (g * 128 + 64 + lane) * 4);
#pragma unroll
                for (int p = 1; p < W; ++p) {
                    x += *(const f32x4_t*)(smem + p * AP_BWD_WAVE + (g * 128 + lane) * 4);
                    xg4 += *(const f32x4_t*)(smem + p * AP_BWD_WAVE + (g * 128 + 64 + lane) * 4);
                }
                put(g, x, xg4);
            }
        }
        sample_sync<W>();
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            if (128 * (w + W * i) >= r) continue;
            const float2 ki = in_loop(tk[i]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float s = ((e ? ki.y : ki.x) - R.kc) * R.iHk;
                int p = (int)((s + 1.f) * (0.5f * (float)n));
                p = p < 0 ? 0 : (p < n ? p : n - 1);
                const int pl = p - 16 * g0;
                const bool mine = pl >= 0 && pl < 16 * gc;
                const float x = (s - fmaf((float)(2 * p + 1), sh, -1.f)) * xs;
                const float* const cp = coef(mine ? pl : 0);
                float c[24];
#pragma unroll
                for (int u = 0; u < 6; ++u) *(f32x4_t*)(c + 4 * u) = *(const f32x4_t*)(cp + 4 * u);
                const float dk = (e ? tv[i].y : tv[i].x) * horner(c, x) - horner(c + 8, x);
                const float dv = beta * (e ? tg[i].y : tg[i].x) + horner(c + 16, x);
                if (mine) {
                    if (e) { c1[i].y = dk; c3[i].y = dv; }
                    else { c1[i].x = dk; c3[i].x = dv; }
                }
            }
        }
        // the next sweep's tiles overwrite polynomials that other waves of the sample still read
        if (W > 1 && g0 + AP_G < ng) __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int j = 128 * (w + W * i) + 2 * lane;
        if (j >= r) continue;
        *(uint32_t*)(gp + j) = pack_bf16x2(c3[i].x, c3[i].y);
        *(uint32_t*)(gp + 2 * r + j) = pack_bf16x2(c1[i].x, c1[i].y);
    }
}

// Direct column sums of one sample. They run on the matrix cores with K over rows:
// the exponent arguments come out of v_mfma_f32_32x32x8_f16 with the row records as A
// and the key fragments as B (the forward's product with its operands swapped, so each
// e_ij is computed exactly as in the forward), which leaves lane l holding e of key
// l % 32 for 16 rows of a 32-row block: the B operands of two v_mfma_f32_16x16x32_f16
// against Y^T (rows: a hi, a lo, a o hi, a o lo, go/Z hi, lo), keys n and n + 16 in
// output slots 0-7 and 8-15 (frag32).
// A sample's waves split its keys (16 ATT_BWD_KT at a time); every wave runs over all rows.
template <typename T, int W, int KB, int KT>
__device__ __forceinline__ void attn_bwd_direct(int r, int rpad, float alpha, float beta, float inv_tau,
                                                const float* __restrict__ pv, const float* __restrict__ so,
                                                const float* __restrict__ gh, float* sk, int lane, int wave,
                                                T* __restrict__ gp) {
    // sk: [rpad] keys
    const int w = W == 1 ? 0 : wave;
    float2* scm = (float2*)(sk + rpad);                      // [rpad] row constants
    _Float16* sy = (_Float16*)(scm + rpad);                  // Y^T, 6 rows
    float* slots = sk + attn_bwd_sample_floats(rpad);
    float* slot = slots + w * attn_bwd_wave_floats();
    const int ldy = rpad;
    const float* pq = pv + r;
    const float* pk = pv + 2 * r;
    constexpr int KPL = 4 * KB;      // keys (and rows) per lane: 64 KPL >= rpad
    constexpr int RPW = KPL / W;     // rows per lane of this wave's share: 64 (s W + w) + lane
    float kr[KPL];
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        const int j = 64 * u + lane;
        kr[u] = pk[j < r ? j : r - 1];
    }
#pragma unroll
    for (int u = 0; u < KPL; ++u)
        if (64 * u + lane >= r) kr[u] = 0.f;
    float kmin, kmax;
    key_range<KPL>(kr, r, lane, kmin, kmax);
    // this wave's rows: the forward's statistics, dq, and the column-sum coefficients
    float qr[RPW], ghr[RPW], orr[RPW], zr[RPW], dr[RPW];
#pragma unroll
    for (int s = 0; s < RPW; ++s) {
        const int i = 64 * (s * W + w) + lane, ic = i < r ? i : r - 1;
        qr[s] = pq[ic];
        ghr[s] = gh[ic];
        orr[s] = so[ic];
        zr[s] = so[r + ic];
        dr[s] = so[2 * r + ic];
    }
    float ca[RPW], cb[RPW], cg[RPW], c[RPW], m[RPW];
    float big = fmaxf(fabsf(kmin), fabsf(kmax)), ma = 0.f, mb = 0.f, mc = 0.f;
#pragma unroll
    for (int s = 0; s < RPW; ++s) {
        const int i = 64 * (s * W + w) + lane;
        const bool ok = i < r;
        const float q = ok ? qr[s] : 0.f, go = ok ? alpha * ghr[s] : 0.f;
        const float rz = ok && zr[s] != 0.f ? __builtin_amdgcn_rcpf(zr[s]) : 0.f;
        if (ok) st<T>::store(gp + r + i, go * inv_tau * dr[s]);
        ca[s] = go * q * rz * inv_tau;
        cb[s] = ca[s] * orr[s];
        cg[s] = go * rz;
        c[s] = q * (LOG2E * inv_tau);
        m[s] = -(c[s] * (c[s] >= 0.f ? kmax : kmin));
        if (ok) big = fmaxf(big, fmaxf(fabsf(c[s]), fabsf(m[s])));
        ma = fmaxf(ma, fabsf(ca[s]));
        mb = fmaxf(mb, fabsf(cb[s]));
        mc = fmaxf(mc, fabsf(cg[s]));
    }
    big = wave_max(big);
    ma = wave_max(ma);
    mb = wave_max(mb);
    mc = wave_max(mc);
    if (W > 1) {  // maxima over the sample's rows
        if (lane == 0) {
            slot[0] = big;
            slot[1] = ma;
            slot[2] = mb;
            slot[3] = mc;
        }
        __syncthreads();
        big = sample_max<W>(slots, attn_bwd_wave_floats(), 0);
        ma = sample_max<W>(slots, attn_bwd_wave_floats(), 1);
        mb = sample_max<W>(slots, attn_bwd_wave_floats(), 2);
        mc = sample_max<W>(slots, attn_bwd_wave_floats(), 3);
    }
    const bool fast = uniform_f(big) < ATT_F16_SAFE;  // the forward's decision
    const float as = uniform_f(pow2_ceil(ma)), bs = uniform_f(pow2_ceil(mb)), cs = uniform_f(pow2_ceil(mc));
    const float ias = 1.0f / as, ibs = 1.0f / bs, ics = 1.0f / cs;  // exact: powers of two
#pragma unroll
    for (int u = 0; u < KPL; ++u) {
        const int j = 64 * u + lane;
        if (j < rpad && u % W == w) sk[j] = kr[u];
    }
#pragma unroll
    for (int s = 0; s < RPW; ++s) {
        const int i = 64 * (s * W + w) + lane;
        if (i < rpad) {
            if (fast) *(f16x4_t*)(scm + i) = row_rec(c[s], m[s]);
            else scm[i] = make_float2(c[s], m[s]);
            put_pair(sy, ldy, 0, i, ca[s] * ias);
            put_pair(sy, ldy, 2, i, cb[s] * ibs);
            put_pair(sy, ldy, 4, i, cg[s] * ics);
            sy[xoff(6, i, ldy)] = (_Float16)0.f;
            sy[xoff(7, i, ldy)] = (_Float16)0.f;
        }
    }
    sample_sync<W>();

    const int g = lane >> 4, n = lane & 15;
    // Fast path: 32-key blocks. Arguments of 32 rows x 32 keys from one 32x32x8 MFMA
    // (row records as A, key records as B: lane l gets key l % 32), then two column
    // sums per block whose output lane (g4, n) holds quantities 4 (g4 & 1) .. +3 of
    // key n + 16 (g4 / 2).
    auto keys32 = [&]() {
        constexpr int KB2 = KT / 2;
        for (int j0 = 16 * KT * w; j0 < rpad; j0 += 16 * KT * W) {
            f16x4_t kf[KB2];
            float ev[KB2], eg[KB2];
#pragma unroll
            for (int q = 0; q < KB2; ++q) {
                const int jl = j0 + 32 * q + (lane & 31), jp = jl < rpad ? jl : rpad - 1;
                kf[q] = key_frag(sk[jp], lane >> 5);
                const int j = j0 + 32 * q + n + 16 * (lane >> 5), jc = j < r ? j : r - 1;
                ev[q] = pv[jc];
                eg[q] = gh[jc];
            }
            f32x4_t col[KB2];
#pragma unroll
            for (int q = 0; q < KB2; ++q) col[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            const f32x16_t z16 = {};
            for (int i0 = 0; i0 < rpad; i0 += 32) {
                const f16x4_t rec = *(const f16x4_t*)(scm + i0 + (lane & 31));
                const f16x8_t y0 = yfrag32(sy, ldy, lane, i0), y1 = yfrag32(sy, ldy, lane, i0 + 16);
                f32x16_t x[KB2];
#pragma unroll
                for (int q = 0; q < KB2; ++q) x[q] = __builtin_amdgcn_mfma_f32_32x32x8f16(rec, kf[q], z16, 0, 0, 0);
#pragma unroll
                for (int q = 0; q < KB2; ++q) {
                    float e0[8], e1[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        e0[u] = __builtin_amdgcn_exp2f(x[q][u]);
                        e1[u] = __builtin_amdgcn_exp2f(x[q][8 + u]);
                    }
                    col[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(y0, __builtin_bit_cast(f16x8_t, pack_e(e0)), col[q], 0, 0, 0);
                    col[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(y1, __builtin_bit_cast(f16x8_t, pack_e(e1)), col[q], 0, 0, 0);
                }
            }
#pragma unroll
            for (int q = 0; q < KB2; ++q) {
                const int j = j0 + 32 * q + n + 16 * (lane >> 5);
                if (j < r) {
                    if (((lane >> 4) & 1) == 0) {
                        const float c1 = (col[q].x + col[q].y) * as, c2 = (col[q].z + col[q].w) * bs;
                        st<T>::store(gp + 2 * r + j, ev[q] * c1 - c2);
                    } else {
                        st<T>::store(gp + j, beta * eg[q] + (col[q].x + col[q].y) * cs);
                    }
                }
            }
        }
    };
    // Slow path (arguments by FMA): 16-key tiles, lane (g, n) holds e of key n for
    // rows 4 g .. +3 and 16 + 4 g .. +3 of each 32-row block.
    auto keys_fma = [&]() {
        for (int j0 = 16 * KT * w; j0 < rpad; j0 += 16 * KT * W) {
            // keys j0 + 16 q + n of this lane (q < KT; past rpad the last key stands in and
            // nothing is stored); their epilogue operands, loaded now
            float kv[KT], ev[KT], eg[KT];
#pragma unroll
            for (int q = 0; q < KT; ++q) {
                const int j = j0 + 16 * q + n, jp = j < rpad ? j : rpad - 1, jc = j < r ? j : r - 1;
                kv[q] = sk[jp];
                ev[q] = pv[jc];
                eg[q] = gh[jc];
            }
            f32x4_t col[KT];
#pragma unroll
            for (int q = 0; q < KT; ++q) col[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            for (int i0 = 0; i0 < rpad; i0 += 32) {
                const f16x8_t ay = xfrag_perm(sy, ldy, n, 6, i0, g);
                u32x4_t e[KT];
                {
                    // rows i0 + 4 g + t and i0 + 16 + 4 g + t (t < 4) of this lane's keys
                    float2 cm[8];
                    *(f32x4_t*)&cm[0] = *(const f32x4_t*)(scm + i0 + 4 * g);
                    *(f32x4_t*)&cm[2] = *(const f32x4_t*)(scm + i0 + 4 * g + 2);
                    *(f32x4_t*)&cm[4] = *(const f32x4_t*)(scm + i0 + 16 + 4 * g);
                    *(f32x4_t*)&cm[6] = *(const f32x4_t*)(scm + i0 + 16 + 4 * g + 2);
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        float ex[8];
#pragma unroll
                        for (int t = 0; t < 8; ++t) ex[t] = __builtin_amdgcn_exp2f(fmaf(cm[t].x, kv[q], cm[t].y));
                        e[q] = pack_e(ex);
                    }
                }
#pragma unroll
                for (int q = 0; q < KT; ++q)
                    col[q] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ay, __builtin_bit_cast(f16x8_t, e[q]), col[q], 0, 0, 0);
            }
            // lanes 0..15: (a hi, a lo, a o hi, a o lo) of key n (+16 q); lanes 16..31: (go/Z hi, lo)
            if (lane < 32) {
#pragma unroll
                for (int q = 0; q < KT; ++q) {
                    const int j = j0 + 16 * q + n;
                    if (j < r) {
                        if (lane < 16) {
                            const float c1 = (col[q].x + col[q].y) * as, c2 = (col[q].z + col[q].w) * bs;
                            st<T>::store(gp + 2 * r + j, ev[q] * c1 - c2);
                        } else {
                            st<T>::store(gp + j, beta * eg[q] + (col[q].x + col[q].y) * cs);
                        }
                    }
                }
            }
        }
    };
    if (fast) keys32();
    else keys_fma();
}

// Writes gP = [gv | gq | gk].
template <typename T, int W, int KB, bool PANEL>
__global__ __launch_bounds__(64 * att_block_waves(W)) __attribute__((amdgpu_waves_per_eu(PANEL ? 3 : 4, 8))) void k_attn_bwd_mfma(
    int64_t B, int r, int rpad, float alpha, float beta, float inv_tau, const float* __restrict__ P, int64_t ldp,
    const float* __restrict__ stats, const float* __restrict__ GH, int64_t ldg, T* __restrict__ GP, int64_t ldgp) {
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int w = W == 1 ? 0 : wave;
    const int64_t b = (int64_t)blockIdx.x * att_block_samples(W) + (W == 1 ? wave : 0);
    if (b >= B) return;  // (one wave per sample only: with W > 1 there are B workgroups)
    const float* pv = P + b * ldp;
    const float* gh = GH + b * ldg;
    const float* so = stats + b * 3 * (int64_t)r;
    T* gp = GP + b * ldgp;
    if constexpr (!PANEL) {
        attn_bwd_direct<T, W, KB, ATT_BWD_KT>(r, rpad, alpha, beta, inv_tau, pv, so, gh, smem + wave * attn_bwd_direct_floats(rpad, 1),
                                  lane, wave, gp);
        return;
    }
    constexpr int TPW = 2 * KB / W;  // 128-entry tiles of the wave
    float2 k[TPW], v[TPW], g[TPW], y[TPW], a[TPW], ao[TPW], gz[TPW];
    {
        float2 o[TPW], z[TPW], d[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int j = 128 * (w + W * i) + 2 * lane;
            v[i] = load_pair(pv, j, r);
            y[i] = load_pair(pv + r, j, r);  // q for now
            k[i] = load_pair(pv + 2 * r, j, r);
            g[i] = load_pair(gh, j, r);
            o[i] = load_pair(so, j, r);
            z[i] = load_pair(so + r, j, r);
            d[i] = load_pair(so + 2 * r, j, r);
        }
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int j = 128 * (w + W * i) + 2 * lane;
            const bool ok = j < r;
            y[i] = pair_or_zero(y[i], ok);
            const float2 go = pair_or_zero(make_float2(alpha * g[i].x, alpha * g[i].y), ok);
            const float rx = z[i].x != 0.f ? __builtin_amdgcn_rcpf(z[i].x) : 0.f;
            const float ry = z[i].y != 0.f ? __builtin_amdgcn_rcpf(z[i].y) : 0.f;
            if (ok) *(uint32_t*)(gp + r + j) = pack_bf16x2(go.x * inv_tau * d[i].x, go.y * inv_tau * d[i].y);
            gz[i] = make_float2(go.x * rx, go.y * ry);
            a[i] = make_float2(gz[i].x * y[i].x * inv_tau, gz[i].y * y[i].y * inv_tau);
            ao[i] = pair_or_zero(make_float2(a[i].x * o[i].x, a[i].y * o[i].y), ok);
        }
    }
    float mx[6] = {-INFINITY, -INFINITY, 0.f, 0.f, 0.f, 0.f};  // -min k, max k, max |q|, |a|, |a o|, |go/Z|
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        if (128 * (w + W * i) + 2 * lane < r) {
            mx[0] = fmaxf(mx[0], fmaxf(-k[i].x, -k[i].y));
            mx[1] = fmaxf(mx[1], fmaxf(k[i].x, k[i].y));
        }
        mx[2] = abs_max2(mx[2], y[i]);
        mx[3] = abs_max2(mx[3], a[i]);
        mx[4] = abs_max2(mx[4], ao[i]);
        mx[5] = abs_max2(mx[5], gz[i]);
    }
    sample_maxima<W>(smem + attn_bwd_panel_floats(W) - 8 * W, wave, lane, mx);
    const ScoreRange R = score_range(mx[0], mx[1], mx[2], inv_tau, r / 4, AP_RHO_BWD);
    if (R.panels) {
        const float cq = LOG2E * inv_tau * R.Hk;
#pragma unroll
        for (int i = 0; i < TPW; ++i) y[i] = make_float2(y[i].x * cq, y[i].y * cq);
        attn_bwd_panels<T, W, TPW>(R, r, beta, k, v, g, y, a, ao, gz, mx[3], mx[4], mx[5], smem, wave, w, lane, gp);
    } else {
        attn_bwd_direct<T, W, KB, ATT_BWD_KT_WIDE>(r, rpad, alpha, beta, inv_tau, pv, so, gh, W == 1 ? smem + wave * AP_BWD_WAVE : smem, lane, wave,
                                  gp);
    }
}

int attn_threads(int r) {
    int t = ((r + 63) / 64) * 64;
    return t > 256 ? 256 : t;
}

}  // namespace

// Waves per sample: one up to rank 256, else four (one workgroup per sample).
static int attn_waves(int rpad) { return rpad <= 16 * ATT_NT ? 1 : 4; }
// tiles computed per wave: the power of two (>= 2) covering the tiles one wave owns
static int attn_tiles(int rpad, int W) {
    const int ntile = rpad / 16;
    const int per = (((ntile + W - 1) / W) + 1) & ~1;
    int nt = 2;
    while (nt < per) nt *= 2;
    return nt;
}

hipError_t launch_attn_fwd(int64_t B, int r, float alpha, float beta, float tau, const void* P, int64_t ldp, void* H,
                           void* H2, bool h2_f16, int64_t ldh, float* stats, int* err, bool bf16, hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (bf16) {
        if (r > 4 * 16 * ATT_NT || !stats) return hipErrorInvalidValue;
        const int rpad = (r + 31) / 32 * 32;
        const int W = attn_waves(rpad);
        const int NT = attn_tiles(rpad, W);
        const int64_t blocks = W == 1 ? (B + 3) / 4 : B;
        const bool panel = r >= AP_MIN_RANK_FWD;
        const size_t lds = sizeof(float) * (size_t)(panel ? attn_fwd_block_floats(rpad, W) : 4 * attn_fwd_direct_floats(rpad, 1));
#define RDCN_AFWD(WV, NTV, KBV, PNL)                                                                                 \
    hipLaunchKernelGGL((k_attn_fwd_mfma<bf16_t, WV, NTV, KBV, PNL>), dim3((unsigned)blocks),                            \
                       dim3(64 * att_block_waves(WV)), lds, s, B, r, rpad, alpha, beta, 1.0f / tau, (const float*)P,   \
                       ldp, (bf16_t*)H, H2, ldh, h2_f16, stats, err)
        if (!panel) {
            if (NT == 2) RDCN_AFWD(1, 2, 1, false);
            else if (NT == 4) RDCN_AFWD(1, 4, 1, false);
            else RDCN_AFWD(1, 8, 1, false);
        } else if (W == 1) {
            if (NT == 8) RDCN_AFWD(1, 8, 1, true);
            else RDCN_AFWD(1, 16, 1, true);
        } else if (NT == 8) {
            RDCN_AFWD(4, 8, 2, true);
        } else {
            RDCN_AFWD(4, 16, 4, true);
        }
#undef RDCN_AFWD
        return hipGetLastError();
    }
    if (h2_f16) return hipErrorInvalidValue;  // float models have no f16 activations
    const size_t lds = sizeof(float) * (2 * (size_t)r + 32);
    const int th = attn_threads(r);
    hipLaunchKernelGGL(k_attn_fwd<float>, dim3((unsigned)B), dim3(th), lds, s, B, r, alpha, beta, 1.0f / tau,
                       (const float*)P, ldp, (float*)H, (float*)H2, ldh);
    return hipGetLastError();
}

hipError_t launch_attn_bwd(int64_t B, int r, float alpha, float beta, float tau, const void* P, int64_t ldp,
                           const float* stats, const float* GH, int64_t ldg, void* GP, int64_t ldgp, bool bf16,
                           hipStream_t s) {
    if (B == 0) return hipSuccess;
    if (bf16) {
        if (r > 4 * 16 * ATT_NT || !stats) return hipErrorInvalidValue;
        const int rpad = (r + 31) / 32 * 32;
        const int W = attn_waves(rpad);
        const int64_t blocks = W == 1 ? (B + 3) / 4 : B;
        const bool panel = r >= AP_MIN_RANK_BWD;
        const size_t lds = sizeof(float) * (size_t)(panel ? attn_bwd_block_floats(rpad, W) : 4 * attn_bwd_direct_floats(rpad, 1));
#define RDCN_ABWD(WV, KBV, PNL)                                                                                      \
    hipLaunchKernelGGL((k_attn_bwd_mfma<bf16_t, WV, KBV, PNL>), dim3((unsigned)blocks), dim3(64 * att_block_waves(WV)), \
                       lds, s, B, r, rpad, alpha, beta, 1.0f / tau, (const float*)P, ldp, stats, GH, ldg, (bf16_t*)GP, ldgp)
        if (!panel) RDCN_ABWD(1, 1, false);
        else if (W == 1) RDCN_ABWD(1, 1, true);
        else if (rpad <= 512) RDCN_ABWD(4, 2, true);
        else RDCN_ABWD(4, 4, true);
#undef RDCN_ABWD
        return hipGetLastError();
    }
    const size_t lds = sizeof(float) * (7 * (size_t)r + 32);
    const int th = attn_threads(r);
    hipLaunchKernelGGL(k_attn_bwd<float>, dim3((unsigned)B), dim3(th), lds, s, B, r, alpha, beta, 1.0f / tau,
                       (const float*)P, ldp, GH, ldg, (float*)GP, ldgp);
    return hipGetLastError();
}

}  // namespace rdcn
