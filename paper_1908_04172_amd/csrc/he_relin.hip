// The x^2 activation on ciphertexts (Sec. "CryptoNets"; "Square" and "Relinearize" in the paper's table of
// operation runtimes): square a ciphertext and relinearise the result with a special prime (Sec.
// "Homomorphic Encryption": key switching by raising the modulus).  The ciphertext lives on limbs
// q_0..q_{l-1}, 1 <= l <= L-1; the context's last limb is the special prime P.  Working tensors have l+1
// limb positions: q_0..q_{l-1}, then P.  With (d0, d1, d2) = (c0^2, 2 c0 c1, c1^2) slot-wise, four launches:
//   1. d2 and its inverse NTT in one kernel (the transform kernel squares the rows it loads): row j then holds the
//      coefficients of [d2]_{q_j} in [0, q_j), RNS digit j; the NTT-form d2 goes to its place among the digits;
//   2. every digit re-reduced modulo the other q_i and P and transformed under that limb: the transform kernel in
//      its digit-expansion form, l * l rows written from l rows read;
//   3. acc_k = P * d_k + sum_j digit_j * evk[j][k], k = 0, 1, on all l+1 limbs (d_k formed from c0, c1 on the spot);
//   4. division of acc by P with rounding: Eq. (2) with P as the dropped limb, the rescale kernel as it is.  P * d_k is
//      an exact multiple of P, so round(acc / P) = d_k + round(sum / P): the relinearised ciphertext, with no
//      addition of its own.
#include <algorithm>

#include "he_internal.h"

namespace {

// step 3: one thread = one slot of one limb position, both components, for a run of ciphertexts
// (L = l + 1 limb positions; `lt` has the special prime's constants at position l, and `p_mod` its residues modulo
// the other limbs; the key is the top-level one, [..][2][key_limbs][N], in which the special prime is limb
// key_limbs - 1)
// What bounds it: the digits, read once, and the two sums, written once.  The slot's 2 l key residues stay in registers
// for the whole run of ciphertexts (read for every one of them they were as many bytes again as digits and sums
// together, out of the caches), and the sums are MacAcc ones, of which P * d_k is one more term: four multiply-adds per
// product and one reduction per sum.  256 ciphertexts, seven limbs and P, N = 2^14 (2.9 GB): 767 -> 574 us.  The digits are
// read past the caches (the whole square of 200 ciphertexts, four limbs and P, N = 2^13: 408 -> 391 us; of 60 at 2^14 262 -> 249),
// at every size: with 125 to 280 MiB of them that is 2 to 6 % of the square (30 ciphertexts, seven limbs and P, 2^14, 295 -> 279), with
// 90 MiB and less neither way is faster (37 sizes from 1 ciphertext on, all within 0.8 %), with 420 and 700 MiB it is 1 % at most.
// A run of one ciphertext has nothing to keep the key for, and holding it only costs wavefronts (186 registers at l = 15):
// such launches read it term by term (eight ciphertexts at N = 2^13, l = 15: 52 -> 34 us; l = 10: 24 -> 20).
struct SpecialPrimeResidues {
    u64 r[HE_MAX_LIMBS], r_shoup[HE_MAX_LIMBS];
};
constexpr u32 KEY_WORKGROUPS = 8192;  // a launch is cut into at least so many workgroups while there are ciphertexts to cut

// the two sums of a slot
struct KeySums {
    MacAcc a0, a1;
    u32 f = 0, r = 0;
    __device__ __forceinline__ KeySums() {
        acc_clear(a0);
        acc_clear(a1);
    }
    // += x * (w0, w1), all in two pieces
    __device__ __forceinline__ void add(u64 x, u32 w0a, u32 w0b, u32 w1a, u32 w1b, const LimbConst& c) {
        if (r >= c.reduce_every) {
            acc_restart(a0, c);
            acc_restart(a1, c);
            f = r = 0;
        } else if (f >= c.fold_every) {
            acc_fold(a0, c);
            acc_fold(a1, c);
            f = 0;
        }
        ++f;
        ++r;
        u32 xa, xb;
        split_operand(x, c, xa, xb);
        acc_mac(a0, xa, xb, w0a, w0b);
        acc_mac(a1, xa, xb, w1a, w1b);
    }
    __device__ __forceinline__ void add(u64 x, u64 w0, u64 w1, const LimbConst& c) {
        u32 w0a, w0b, w1a, w1b;
        split_operand(w0, c, w0a, w0b);
        split_operand(w1, c, w1a, w1b);
        add(x, w0a, w0b, w1a, w1b, c);
    }
};

// where a thread is: its slot, its limb position and the run of ciphertexts
struct KeyPlace {
    size_t k;
    u32 limb, first, end, key_limb;
    __device__ __forceinline__ KeyPlace(u32 l, u32 key_limbs, u32 N, u32 n, u32 per_wg) {
        u32 b = blockIdx.x;
        k = (size_t)(b % (N / 256)) * 256 + threadIdx.x;
        b /= N / 256;
        limb = b % (l + 1);
        first = b / (l + 1) * per_wg;
        end = min(n, first + per_wg);
        key_limb = limb == l ? key_limbs - 1 : limb;
    }
};

template <int l>
__global__ void __launch_bounds__(256) key_product_kernel(LimbTable lt, SpecialPrimeResidues p_mod, u32 key_limbs, u32 N, const u64* digits,
                                                          u32 n, u32 per_wg, const u64* evk, const u64* ct, u64* acc) {
    constexpr u32 L = l + 1;
    const KeyPlace at0(l, key_limbs, N, n, per_wg);
    const size_t k = at0.k;
    const u32 limb = at0.limb, key_limb = at0.key_limb;
    const LimbConst& c = lt.c[limb];
    u32 ka[2][l], kb[2][l];
#pragma unroll
    for (u32 j = 0; j < l; j++)
#pragma unroll
        for (u32 i = 0; i < 2; i++) split_operand(evk[((size_t)(j * 2 + i) * key_limbs + key_limb) * N + k], c, ka[i][j], kb[i][j]);
    for (u32 at = at0.first; at < at0.end; at++) {
        u64 d[l], c0 = 0, c1 = 0;
#pragma unroll
        for (u32 j = 0; j < l; j++) d[j] = __builtin_nontemporal_load(&digits[(((size_t)at * l + j) * L + limb) * N + k]);
        if (limb < l) {
            c0 = ct[(((size_t)at * 2) * l + limb) * N + k];
            c1 = ct[(((size_t)at * 2 + 1) * l + limb) * N + k];
        }
        KeySums s;
#pragma unroll
        for (u32 j = 0; j < l; j++) s.add(d[j], ka[0][j], kb[0][j], ka[1][j], kb[1][j], c);
        // + P * (c0^2, 2 c0 c1); modulo P itself that is zero
        if (limb < l) s.add(shoup_mul(c0, p_mod.r[limb], p_mod.r_shoup[limb], c.q), c0, add_mod(c1, c1, c.q), c);
        acc[(((size_t)at * 2) * L + limb) * N + k] = acc_reduce(s.a0, c);
        acc[(((size_t)at * 2 + 1) * L + limb) * N + k] = acc_reduce(s.a1, c);
    }
}

// runs of one ciphertext, any l
__global__ void __launch_bounds__(256) key_product_single_kernel(LimbTable lt, SpecialPrimeResidues p_mod, u32 l, u32 key_limbs, u32 N,
                                                                 const u64* digits, u32 n, const u64* evk, const u64* ct, u64* acc) {
    const KeyPlace at0(l, key_limbs, N, n, 1);
    const size_t k = at0.k, at = at0.first;
    const u32 limb = at0.limb, key_limb = at0.key_limb, L = l + 1;
    const LimbConst& c = lt.c[limb];
    KeySums s;
    for (u32 j = 0; j < l; j++) {
        const u64* key = evk + ((size_t)j * 2 * key_limbs + key_limb) * N + k;
        s.add(digits[((at * l + j) * L + limb) * N + k], key[0], key[(size_t)key_limbs * N], c);
    }
    if (limb < l) {
        const u64 c0 = ct[(at * 2 * l + limb) * N + k], c1 = ct[((at * 2 + 1) * l + limb) * N + k];
        s.add(shoup_mul(c0, p_mod.r[limb], p_mod.r_shoup[limb], c.q), c0, add_mod(c1, c1, c.q), c);
    }
    acc[(at * 2 * L + limb) * N + k] = acc_reduce(s.a0, c);
    acc[((at * 2 + 1) * L + limb) * N + k] = acc_reduce(s.a1, c);
}

template <int l>
void launch_key_product(u32 l_wanted, const LimbTable& lt, const SpecialPrimeResidues& p_mod, u32 key_limbs, u32 N, const u64* digits, u32 n,
                        const u64* evk, const u64* ct, u64* acc, hipStream_t s) {
    if constexpr (l < HE_MAX_LIMBS) {
        if (l != l_wanted) return launch_key_product<l + 1>(l_wanted, lt, p_mod, key_limbs, N, digits, n, evk, ct, acc, s);
        const u32 rows = N / 256 * (l + 1);
        const u32 runs = std::min(n, (KEY_WORKGROUPS + rows - 1) / rows), per_wg = (n + runs - 1) / runs;
        const dim3 grid(rows * ((n + per_wg - 1) / per_wg)), block(256);
        if (per_wg == 1)
            hipLaunchKernelGGL(key_product_single_kernel, grid, block, 0, s, lt, p_mod, l, key_limbs, N, digits, n, evk, ct, acc);
        else
            hipLaunchKernelGGL((key_product_kernel<l>), grid, block, 0, s, lt, p_mod, key_limbs, N, digits, n, per_wg, evk, ct, acc);
    }
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

size_t square_relin_workspace(const he_ctx* ctx, u32 l, u32 n) {
    const size_t row = (size_t)ctx->N * sizeof(u64), L = (size_t)l + 1;
    return align256(n * l * row) + align256(n * l * L * row) + align256(n * 2 * L * row);
}

int launch_square_relin(he_ctx* ctx, u32 l, const u64* ct_in, u32 n, const u64* evk, u64* ct_out, void* workspace, hipStream_t s) {
    const u32 L = l + 1, N = ctx->N;  // limb positions of the working tensors: q_0..q_{l-1}, P
    const size_t row = (size_t)N * sizeof(u64);
    char* ws = (char*)workspace;
    u64* d2 = (u64*)ws;
    ws += align256((size_t)n * l * row);
    u64* digits = (u64*)ws;
    ws += align256((size_t)n * l * L * row);
    u64* acc = (u64*)ws;
    const size_t b3 = ((size_t)n * L * N + 255) / 256;
    if (b3 > 0x7FFFFFFFull || (u64)n * l > 0x0FFFFFFFull) return HE_ERR_RANGE;
    LimbTable lt = ctx->limbs;
    lt.c[l] = ctx->limbs.c[ctx->L - 1];  // the special prime at the last position
    SpecialPrimeResidues p_mod = {};
    for (u32 i = 0; i < l; ++i) {
        p_mod.r[i] = ctx->q[ctx->L - 1] % ctx->q[i];
        p_mod.r_shoup[i] = (u64)(((u128)p_mod.r[i] << 64) / ctx->q[i]);
    }
    int rc;
    if ((rc = launch_ntt_square(ctx, l, ct_in, d2, digits, n, s)) != HE_OK) return rc;
    if ((rc = launch_ntt_spread(ctx, L, d2, digits, n * l, l, s)) != HE_OK) return rc;
    launch_key_product<1>(l, lt, p_mod, ctx->L, N, digits, n, evk, ct_in, acc, s);
    HE_HIP(hipGetLastError());
    return launch_rescale_drop(ctx, L, ctx->L - 1, acc, ct_out, n, s);
}
