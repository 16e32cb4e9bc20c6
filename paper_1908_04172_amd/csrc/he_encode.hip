// General CKKS encoding (Alg. 1) and its inverse for gfx950: N/2 complex slots -> the integer polynomial whose values
// at the roots r_k = exp(i*pi*(2k+1)/N), k < N/2, are scale*z_k (and the conjugates at the conjugate
// roots) -> residues per limb.  The forward NTT of the rows follows as a separate launch.
//
// The interpolation is a complex FFT of half the ring size.  Half of the 2N-th roots of unity, those
// with exponent 1 mod 4, satisfy r^(N/2) = i, so on them m(r) = sum_{j < N/2} (m_j + i*m_{j+N/2}) r^j:
// the N real coefficients are the real and imaginary parts of the N/2 complex numbers
//     w_j = xi^-j * (2/N) * sum_kappa z'_kappa * e^(-2 pi i kappa j / (N/2)),   xi = exp(i*pi/N),
// where z'_kappa is the value wanted at xi^(4 kappa + 1): slot 2*kappa itself while 4 kappa + 1 < N,
// otherwise the conjugate of slot N - 2*kappa - 1 (whose own root is the conjugate of that one).
// One workgroup per vector, eight complex values per thread in registers, radix 2, decimation in frequency: three
// stages at a time on registers (a pass), then the values are regrouped through the LDS (N/2 complex doubles = 8N
// bytes) for the next pass.  What bounds these kernels is the chain of stages of one workgroup: with a trip through the
// LDS and a barrier per stage an encoding of 784 vectors at N = 2^13 took 123 us and a decoding of 100 vectors 52 us, with
// three stages per trip they take 68 and 31 us (butterflies, their order and their twiddles are the same, and so are the
// results, bit for bit).
#include "he_internal.h"

namespace {

struct cplx {
    double re, im;
};

// (which product is rounded first is spelled out: the encoder's coefficients are rounded to integers, so its doubles must
// not depend on how the compiler contracts the expression in its context)
__device__ __forceinline__ cplx cmul(cplx a, cplx b) {
    return cplx{__builtin_fma(a.re, b.re, -(a.im * b.im)), __builtin_fma(a.im, b.re, a.re * b.im)};
}

// A value as it is: nothing is contracted across it, so that what the LDS held between two stages before they ran on
// registers is rounded as it was there.
__device__ __forceinline__ cplx rounded(cplx v) {
    asm("" : "+v"(v.re));
    asm("" : "+v"(v.im));
    return v;
}

// The FFT of n = N/2 points on T = n/8 threads.  Stage s pairs indices that differ in bit LOGn-1-s; pass P runs stages
// 3P .. 3P+2 and owns those three index bits, the last pass the lowest three, of which it runs what stages are left.
template <int LOGN>
struct Fft {
    static constexpr u32 N = 1u << LOGN, n = N / 2, T = N / 16;
    static constexpr int LOGn = LOGN - 1, NPASS = (LOGn + 2) / 3;
    static constexpr int low(int P) { return P < NPASS - 1 ? LOGn - 3 * (P + 1) : 0; }  // lowest of the pass's bits
    __device__ static u32 index(int P, u32 tid, u32 e) {
        const u32 lo = tid & ((1u << low(P)) - 1);
        return ((tid ^ lo) << 3) | (e << low(P)) | lo;
    }
    // where the LDS holds an index while the values are regrouped, and in the last exchange: a wide access is served
    // for eight lanes at a time, and the eight neighbouring lanes of every pattern used here differ in the low three bits
    __device__ static u32 slot(u32 i) { return i ^ ((i >> 3) & 7u); }
    __device__ static u32 last_slot(u32 i) { return i ^ ((i >> (LOGn - 6)) & 7u); }
};

// pass P of the transform with twiddles `tw` (CONJ: their conjugates)
template <int LOGN, int P, bool CONJ>
__device__ __forceinline__ void fft_pass(cplx (&v)[8], const cplx* tw, cplx* buf, u32 tid) {
    using F = Fft<LOGN>;
    constexpr int low = F::low(P), S0 = 3 * P, S1 = P < F::NPASS - 1 ? S0 + 3 : F::LOGn;  // its stages
    if constexpr (P > 0) {
        if constexpr (P > 1) __syncthreads();
#pragma unroll
        for (u32 e = 0; e < 8; e++) buf[F::slot(F::index(P - 1, tid, e))] = v[e];
        __syncthreads();
#pragma unroll
        for (u32 e = 0; e < 8; e++) v[e] = buf[F::slot(F::index(P, tid, e))];
    }
#pragma unroll
    for (int s = S0; s < S1; s++) {
        const int bit = F::LOGn - 1 - s - low;  // of the register number
        const u32 lo = tid & ((1u << low) - 1);
#pragma unroll
        for (u32 r = 0; r < (1u << bit); r++) {
            cplx w = tw[((r << low) | lo) << s];
            if (CONJ) w.im = -w.im;
#pragma unroll
            for (u32 e = r; e < 8; e += 2u << bit) {
                const cplx a = v[e], c = v[e | (1u << bit)];
                v[e] = cplx{a.re + c.re, a.im + c.im};
                v[e | (1u << bit)] = rounded(cmul(cplx{a.re - c.re, a.im - c.im}, w));
            }
        }
    }
}

template <int LOGN, bool CONJ>
__device__ __forceinline__ void fft(cplx (&v)[8], const cplx* tw, cplx* buf, u32 tid) {
    using F = Fft<LOGN>;
    static_assert(F::NPASS >= 3 && F::NPASS <= 5, "three to five passes");
    fft_pass<LOGN, 0, CONJ>(v, tw, buf, tid);
    fft_pass<LOGN, 1, CONJ>(v, tw, buf, tid);
    fft_pass<LOGN, 2, CONJ>(v, tw, buf, tid);
    if constexpr (F::NPASS > 3) fft_pass<LOGN, 3, CONJ>(v, tw, buf, tid);
    if constexpr (F::NPASS > 4) fft_pass<LOGN, 4, CONJ>(v, tw, buf, tid);
}

template <int LOGN>
__global__ void __launch_bounds__((1 << LOGN) / 16, 4)
encode_vector_kernel(LimbTable lt, u32 limbs, const cplx* slots, double scale, const cplx* fft_tw, const cplx* twist,
                     u64* out) {
    using F = Fft<LOGN>;
    constexpr u32 N = F::N, n = F::n, T = F::T, LOGn = F::LOGn;
    extern __shared__ cplx buf[];
    const u32 tid = threadIdx.x;
    const cplx* z = slots + (size_t)blockIdx.x * n;
    const double f = scale / (double)n;
    cplx w[8];
#pragma unroll
    for (u32 e = 0; e < 8; e++) {
        const u32 kappa = F::index(0, tid, e);
        cplx v;
        if (4 * kappa + 1 < N) {
            v = z[2 * kappa];
        } else {
            v = z[N - 2 * kappa - 1];
            v.im = -v.im;
        }
        w[e] = rounded(cplx{v.re * f, v.im * f});
    }
    fft<LOGN, false>(w, fft_tw, buf, tid);
    // position pos holds the output of index bitrev(pos): twist it, then put it where it belongs
    __syncthreads();
#pragma unroll
    for (u32 e = 0; e < 8; e++) {
        const u32 at = __brev(F::index(F::NPASS - 1, tid, e)) >> (32 - LOGn);
        buf[F::last_slot(at)] = cmul(w[e], twist[at]);
    }
    __syncthreads();
    // coefficient j = round(Re w_j), coefficient j + N/2 = round(Im w_j); residues of every limb
    u64* rows = out + (size_t)blockIdx.x * limbs * N;
    for (u32 j = tid; j < n; j += T) {
        const cplx v = buf[F::last_slot(j)];
        const RoundedValue lo = round_value(v.re), hi = round_value(v.im);
        for (u32 i = 0; i < limbs; i++) {
            rows[(size_t)i * N + j] = residue_of(lo, lt.c[i]);
            rows[(size_t)i * N + n + j] = residue_of(hi, lt.c[i]);
        }
    }
}

template <int LOGN>
int launch_t(he_ctx* ctx, u32 limbs, const double* slots, u32 n, double scale, u64* out, hipStream_t s) {
    constexpr u32 N = 1u << LOGN;
    const size_t lds = (size_t)N * 8;
    static std::atomic<uint32_t> lds_allowed{0};
    if (int rc = allow_dynamic_lds((const void*)encode_vector_kernel<LOGN>, lds, ctx->device, lds_allowed)) return rc;
    hipLaunchKernelGGL((encode_vector_kernel<LOGN>), dim3(n), dim3(N / 16), lds, s, ctx->limbs, limbs,
                       reinterpret_cast<const cplx*>(slots), scale, reinterpret_cast<const cplx*>(ctx->fft_tw),
                       reinterpret_cast<const cplx*>(ctx->twist), out);
    HE_HIP(hipGetLastError());
    return HE_OK;
}

// ---------------------------------------------------------------------------------------------
// Decoding: the inverse map.  Per coefficient the residues are lifted to the integer of smallest
// magnitude by Garner's mixed-radix form  x = v_0 + v_1 q_0 + v_2 q_0 q_1 + ...  (v_i < q_i, modular
// arithmetic only); x > Q/2 is decided exactly by comparing digits with those of floor(Q/2), and then
// Q - x is formed digit by digit, so the conversion to double (Horner, from the top digit) never
// subtracts large numbers.  The slots are the values of the polynomial at the slot roots: the same
// half-size FFT with the opposite sign, preceded by the twist xi^j.
struct GarnerInv {
    u64 inv, inv_shoup;  // q_k^-1 mod q_i and its Shoup companion, at [i * HE_MAX_LIMBS + k]
};

// (LMAX: a compile-time bound on `limbs`, 8 or HE_MAX_LIMBS: the unrolled loops and the digit registers are that many)
template <int LMAX>
__device__ __forceinline__ double lift_centred(const u64* col, size_t limb_stride, u32 limbs, const LimbTable& lt,
                                               const GarnerInv* g, const u64* half_digits) {
    u64 v[LMAX];
#pragma unroll
    for (u32 i = 0; i < (u32)LMAX; i++) {
        if (i < limbs) {
            const LimbConst& c = lt.c[i];
            u64 t = col[i * limb_stride];
#pragma unroll
            for (u32 k = 0; k < i; k++) {
                const u64 vk = v[k] < c.q ? v[k] : reduce64(v[k], c);
                t = shoup_mul(sub_mod(t, vk, c.q), g[i * HE_MAX_LIMBS + k].inv, g[i * HE_MAX_LIMBS + k].inv_shoup, c.q);
            }
            v[i] = t;
        }
    }
    bool above = false, decided = false;
#pragma unroll
    for (int i = LMAX - 1; i >= 0; i--) {
        if ((u32)i < limbs && !decided && v[i] != half_digits[i]) {
            above = v[i] > half_digits[i];
            decided = true;
        }
    }
    if (above) {  // digits of Q - x = (Q - 1 - x) + 1
        bool carry = true;
#pragma unroll
        for (u32 i = 0; i < (u32)LMAX; i++) {
            if (i < limbs) {
                u64 d = lt.c[i].q - 1 - v[i];
                if (carry) {
                    d += 1;
                    carry = d == lt.c[i].q;
                    if (carry) d = 0;
                }
                v[i] = d;
            }
        }
    }
    double acc = 0.0;
#pragma unroll
    for (int i = LMAX - 1; i >= 0; i--)
        if ((u32)i < limbs) acc = acc * (double)lt.c[i].q + (double)v[i];
    return above ? -acc : acc;
}

template <int LOGN, int LMAX>
__global__ void __launch_bounds__((1 << LOGN) / 16)
decode_vector_kernel(LimbTable lt, u32 limbs, const u64* coef, double inv_scale, const GarnerInv* garner,
                     const u64* half_digits, const cplx* fft_tw, const cplx* twist, cplx* slots) {
    using F = Fft<LOGN>;
    constexpr u32 N = F::N, n = F::n, T = F::T, LOGn = F::LOGn;
    extern __shared__ cplx buf[];
    const u32 tid = threadIdx.x;
    const u64* rows = coef + (size_t)blockIdx.x * limbs * N;
    // (the lift is one loop body, not eight: its results wait in the LDS, each thread's own)
    for (u32 j = tid; j < n; j += T) {
        const double re = lift_centred<LMAX>(rows + j, N, limbs, lt, garner, half_digits) * inv_scale;
        const double im = lift_centred<LMAX>(rows + n + j, N, limbs, lt, garner, half_digits) * inv_scale;
        const cplx tw = twist[j];
        buf[j] = cmul(cplx{re, im}, cplx{tw.re, -tw.im});  // times xi^j
    }
    cplx w[8];
#pragma unroll
    for (u32 e = 0; e < 8; e++) w[e] = buf[F::index(0, tid, e)];
    __syncthreads();
    fft<LOGN, true>(w, fft_tw, buf, tid);
    __syncthreads();
#pragma unroll
    for (u32 e = 0; e < 8; e++) buf[F::last_slot(__brev(F::index(F::NPASS - 1, tid, e)) >> (32 - LOGn))] = w[e];
    __syncthreads();
    // buf[kappa] is the value at xi^(4 kappa + 1): slot 2*kappa, or the conjugate of slot N - 2*kappa - 1
    cplx* z = slots + (size_t)blockIdx.x * n;
    for (u32 k = tid; k < n; k += T) {
        cplx v = buf[F::last_slot((k & 1) ? (N - k - 1) / 2 : k / 2)];
        if (k & 1) v.im = -v.im;
        z[k] = v;
    }
}

template <int LOGN>
int launch_decode_t(he_ctx* ctx, u32 limbs, const u64* coef, u32 n, double scale, double* slots, hipStream_t s) {
    constexpr u32 N = 1u << LOGN;
    const size_t lds = (size_t)N * 8;
    auto launch = [&](auto kernel, std::atomic<uint32_t>& lds_allowed) -> int {
        if (int rc = allow_dynamic_lds((const void*)kernel, lds, ctx->device, lds_allowed)) return rc;
        hipLaunchKernelGGL(kernel, dim3(n), dim3(N / 16), lds, s, ctx->limbs, limbs, coef, 1.0 / scale,
                           reinterpret_cast<const GarnerInv*>(ctx->garner), ctx->half_digits + (size_t)limbs * HE_MAX_LIMBS,
                           reinterpret_cast<const cplx*>(ctx->fft_tw), reinterpret_cast<const cplx*>(ctx->twist),
                           reinterpret_cast<cplx*>(slots));
        HE_HIP(hipGetLastError());
        return HE_OK;
    };
    static std::atomic<uint32_t> lds_allowed_8{0}, lds_allowed_all{0};
    if (limbs <= 8) return launch(decode_vector_kernel<LOGN, 8>, lds_allowed_8);
    return launch(decode_vector_kernel<LOGN, HE_MAX_LIMBS>, lds_allowed_all);
}

}  // namespace

int launch_decode_vector(he_ctx* ctx, u32 limbs, const u64* coef, u32 n, double scale, double* slots, hipStream_t s) {
    switch (ctx->log2N) {
        case 10: return launch_decode_t<10>(ctx, limbs, coef, n, scale, slots, s);
        case 11: return launch_decode_t<11>(ctx, limbs, coef, n, scale, slots, s);
        case 12: return launch_decode_t<12>(ctx, limbs, coef, n, scale, slots, s);
        case 13: return launch_decode_t<13>(ctx, limbs, coef, n, scale, slots, s);
        case 14: return launch_decode_t<14>(ctx, limbs, coef, n, scale, slots, s);
    }
    return HE_ERR_ARG;
}

int launch_encode_vector(he_ctx* ctx, u32 limbs, const double* slots, u32 n, double scale, u64* out, hipStream_t s) {
    switch (ctx->log2N) {
        case 10: return launch_t<10>(ctx, limbs, slots, n, scale, out, s);
        case 11: return launch_t<11>(ctx, limbs, slots, n, scale, out, s);
        case 12: return launch_t<12>(ctx, limbs, slots, n, scale, out, s);
        case 13: return launch_t<13>(ctx, limbs, slots, n, scale, out, s);
        case 14: return launch_t<14>(ctx, limbs, slots, n, scale, out, s);
    }
    return HE_ERR_ARG;
}
