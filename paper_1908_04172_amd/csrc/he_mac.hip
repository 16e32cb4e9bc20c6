// Ciphertext x plaintext multiply-accumulate on the vector ALU (Alg. 7 / Alg. 8 summed over a plan): full-polynomial
// plaintexts, and scalar plaintexts of outputs that share their inputs with no other output.  (Scalar plaintexts of
// groups of outputs run on the matrix cores: he_mac_digits.hip.)
//
// Products are accumulated unreduced (MacAcc) and reduced once at the end (or every LimbConst::reduce_every terms),
// then the bias residue is added on component 0.
#include <algorithm>
#include <type_traits>

#include "he_internal.h"

namespace {

constexpr int MAC_THREADS = 256;
constexpr int GATHER_BLOCKS = 8;

// Weight table of the single outputs: word t of a group's table is the two pieces (wa | wb << 32, see MacAcc) of
// pt[term_pt[off[out0] + t_begin + t]][limb].  Groups with the same plaintext indices share one table.
__global__ void __launch_bounds__(256) gather_weights_kernel(LimbTable lt, const Tile* tiles, const u64* wbase, const u32* owners, u32 n_tables,
                                                             u32 limbs, const u32* off, const u32* term_pt, const u64* pt,
                                                             u64* wtab, u64 tab_words, u64 tab_skip, u32 t_begin, u32 t_end) {
    const u32 table = blockIdx.x / GATHER_BLOCKS, sub = blockIdx.x % GATHER_BLOCKS;
    if (table >= n_tables) return;
    const u32 tile_i = owners[table];
    const Tile tile = tiles[tile_i];
    const u32 first = min(t_begin, tile.n_terms), K = min(t_end, tile.n_terms) - first;
    const u64 total = (u64)K * limbs;
    u64* dst = wtab + (wbase[tile_i] - tab_skip);
    for (u64 i = (u64)sub * blockDim.x + threadIdx.x; i < total; i += (u64)GATHER_BLOCKS * blockDim.x) {
        const u32 limb = (u32)(i / K), t = (u32)(i % K);
        u32 wa, wb;
        split_operand(pt[(size_t)term_pt[off[tile.out0] + first + t] * limbs + limb], lt.c[limb], wa, wb);
        dst[(u64)limb * tab_words + t] = (u64)wa | ((u64)wb << 32);
    }
}

template <int A>
__device__ __forceinline__ void fold_all(MacAcc (&acc)[A], const LimbConst& c) {
#pragma unroll
    for (int g = 0; g < A; g++) acc_fold(acc[g], c);
}

template <int A>
__device__ __forceinline__ void restart_all(MacAcc (&acc)[A], const LimbConst& c) {
#pragma unroll
    for (int g = 0; g < A; g++) {
        acc_restart(acc[g], c);
        __builtin_amdgcn_sched_barrier(0);  // one reduction at a time: keeps its temporaries few
    }
}

// Called between runs of terms: reduce when `reduce_period` terms have gone by since the last
// reduction, else fold when `fold_period` terms have gone by since the last fold.
template <int A>
__device__ __forceinline__ void housekeeping(MacAcc (&acc)[A], u32& f, u32& r, u32 fold_period, u32 reduce_period,
                                             const LimbConst& c) {
    if (r >= reduce_period) {
        restart_all<A>(acc, c);
        r = 0;
        f = 0;
    } else if (f >= fold_period) {
        fold_all<A>(acc, c);
        f = 0;
    }
}

// Outputs that share their inputs with no other output (one multiply per output is the extreme
// case: a plain Alg. 8 call over a tensor).  There is little arithmetic per byte here, so the kernel
// is shaped for the memory system instead: a thread handles SL pairs of adjacent residues (16-byte
// accesses, SL independent loads in flight), a workgroup 512*SL residues of one row.
// WAVES: the wavefronts per SIMD, no more and no fewer.  The registers allow five, which longer sums want; up to two terms the
// fifth only adds rows to what the memory is working on at once.  N = 2^14, L = 4, four and five (the launch): one term
// of 500 ciphertexts 196 and 204 us, two terms of 300 149 and 151, four 210 and 200, nine 285 and 252.
// STREAM: the stores go past the caches (mac_singles_stream).
template <int SL, int WAVES, bool STREAM>
__global__ void __launch_bounds__(MAC_THREADS) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES)))
mac_scalar_single_kernel(LimbTable lt, u32 limbs, u32 N, const Tile* tiles, u32 n_tiles, const u64* wbase, const u32* term_ct,
                         const u64* wtab, u64 tab_words, u64 tab_skip, u32 t_begin, u32 t_end, const u64* ct_in, const u64* bias, u64* out,
                         u32 accumulate) {
    const u32 per_block = MAC_THREADS * 2 * SL;
    const u32 blocks_per_row = N / per_block;
    u32 b = blockIdx.x;
    const u32 part = b % blocks_per_row; b /= blocks_per_row;
    const u32 tile_i = b % n_tiles; b /= n_tiles;
    const u32 comp = b & 1;
    const u32 limb = b >> 1;
    const Tile tile = tiles[tile_i];
    const LimbConst& c = lt.c[limb];
    const size_t ct_stride = (size_t)2 * limbs * N;
    const size_t row_off = ((size_t)comp * limbs + limb) * N + (size_t)part * per_block;
    const u32 first = min(t_begin, tile.n_terms), K = min(t_end, tile.n_terms) - first;
    const u64* w = wtab + (u64)limb * tab_words + (wbase[tile_i] - tab_skip);
    const u32* tc = term_ct + tile.term0 + first;

    MacAcc acc[SL][2];
#pragma unroll
    for (int s = 0; s < SL; s++) { acc_clear(acc[s][0]); acc_clear(acc[s][1]); }
    u32 f = 0, r = 0;
    for (u32 t = 0; t < K; ++t) {
        const u64x2* row = reinterpret_cast<const u64x2*>(ct_in + (size_t)tc[t] * ct_stride + row_off);
        const u64 wv = w[t];
        u64x2 x[SL];
#pragma unroll
        for (int s = 0; s < SL; s++) x[s] = row[s * MAC_THREADS + threadIdx.x];
#pragma unroll
        for (int s = 0; s < SL; s++) {
            u32 xa, xb;
            split_operand(x[s].x, c, xa, xb);
            acc_mac(acc[s][0], xa, xb, (u32)wv, (u32)(wv >> 32));
            split_operand(x[s].y, c, xa, xb);
            acc_mac(acc[s][1], xa, xb, (u32)wv, (u32)(wv >> 32));
        }
        ++f;
        ++r;
        if (t + 1 < K) {
            if (r >= c.reduce_every) {
#pragma unroll
                for (int s = 0; s < SL; s++) { acc_restart(acc[s][0], c); acc_restart(acc[s][1], c); }
                r = 0;
                f = 0;
            } else if (f >= c.fold_every) {
#pragma unroll
                for (int s = 0; s < SL; s++) { acc_fold(acc[s][0], c); acc_fold(acc[s][1], c); }
                f = 0;
            }
        }
    }
    const u32 o = tile.out0;
    const u64 bv = (bias != nullptr && comp == 0) ? bias[(size_t)o * limbs + limb] : 0;
    u64x2* dst = reinterpret_cast<u64x2*>(out + (size_t)o * ct_stride + row_off);
#pragma unroll
    for (int s = 0; s < SL; s++) {
        u64x2 v;
        v.x = add_mod(acc_reduce(acc[s][0], c), bv, c.q);
        v.y = add_mod(acc_reduce(acc[s][1], c), bv, c.q);
        if (accumulate & MAC_ACCUMULATE) {
            const u64x2 old = dst[s * MAC_THREADS + threadIdx.x];
            v.x = add_mod(v.x, old.x, c.q);
            v.y = add_mod(v.y, old.y, c.q);
        }
        if constexpr (STREAM) __builtin_nontemporal_store(v, &dst[s * MAC_THREADS + threadIdx.x]);
        else dst[s * MAC_THREADS + threadIdx.x] = v;
    }
}

// Full-polynomial plaintexts: the plaintext residue differs per slot, is loaded once and used for
// both ciphertext components.  A thread owns two adjacent slots (16-byte accesses) of one limb, for
// G outputs x 2 components: 4*G accumulators.
template <int G>
__global__ void __launch_bounds__(MAC_THREADS)
mac_poly_kernel(LimbTable lt, u32 limbs, u32 N, const Tile* tiles, u32 n_tiles, const u32* off, const u32* term_ct, const u32* term_pt,
                const u64* pt, const u64* ct_in, const u64* bias, u64* out, u32 accumulate) {
    const u32 chunks = N / (2 * MAC_THREADS);
    u32 b = blockIdx.x;  // same order as the scalar kernel: slice, group of outputs, limb
    const u32 chunk = b % chunks; b /= chunks;
    const u32 tile_i = b % n_tiles;
    const u32 limb = b / n_tiles;
    const Tile tile = tiles[tile_i];
    const LimbConst& c = lt.c[limb];
    const u32 n = 2 * (chunk * MAC_THREADS + threadIdx.x);
    const size_t ct_stride = (size_t)2 * limbs * N;
    const size_t comp_stride = (size_t)limbs * N;
    const u64* x_base = ct_in + (size_t)limb * N + n;
    const u64* p_base = pt + (size_t)limb * N + n;
    const size_t pt_stride = (size_t)limbs * N;
    const u32* tc = term_ct + tile.term0;
    const u32 K = tile.n_terms;
    const u32* tp[G];
#pragma unroll
    for (int g = 0; g < G; g++) tp[g] = term_pt + off[tile.out0 + ((u32)g < tile.count ? g : 0)];

    MacAcc acc[4 * G];  // [output][component][slot]
#pragma unroll
    for (int g = 0; g < 4 * G; g++) acc_clear(acc[g]);
    u32 f = 0, r = 0;
    // The operands of term t + 1 are requested before term t is multiplied: twice the bytes in flight per wave
    // (the kernel is bound by HBM latency times the bytes outstanding).  Outputs beyond the group's count read the
    // first output's plaintexts again (tp[g] points there) and are not stored.
    u64x2 x0, x1, p[G];
    auto request = [&](u32 t, u64x2& a0, u64x2& a1, u64x2 (&w)[G]) {
        const u64* xp = x_base + (size_t)tc[t] * ct_stride;
        a0 = *reinterpret_cast<const u64x2*>(xp);
        a1 = *reinterpret_cast<const u64x2*>(xp + comp_stride);
#pragma unroll
        for (int g = 0; g < G; g++) {
            // read once: a non-temporal load keeps it from displacing the reused ciphertext rows in L2
            const u64* src = p_base + (size_t)tp[g][t] * pt_stride;
            w[g].x = __builtin_nontemporal_load(src);
            w[g].y = __builtin_nontemporal_load(src + 1);
        }
    };
    if (K > 0) request(0, x0, x1, p);
    for (u32 t = 0; t < K; t++) {
        u64x2 x0n = x0, x1n = x1, pn[G];
#pragma unroll
        for (int g = 0; g < G; g++) pn[g] = p[g];
        if (t + 1 < K) request(t + 1, x0n, x1n, pn);
        u32 xa[4], xb[4];  // [component][slot]
        split_operand(x0.x, c, xa[0], xb[0]);
        split_operand(x0.y, c, xa[1], xb[1]);
        split_operand(x1.x, c, xa[2], xb[2]);
        split_operand(x1.y, c, xa[3], xb[3]);
#pragma unroll
        for (int g = 0; g < G; g++) {
            u32 pa0, pb0, pa1, pb1;
            split_operand(p[g].x, c, pa0, pb0);
            split_operand(p[g].y, c, pa1, pb1);
            acc_mac(acc[4 * g + 0], xa[0], xb[0], pa0, pb0);
            acc_mac(acc[4 * g + 1], xa[1], xb[1], pa1, pb1);
            acc_mac(acc[4 * g + 2], xa[2], xb[2], pa0, pb0);
            acc_mac(acc[4 * g + 3], xa[3], xb[3], pa1, pb1);
        }
        ++f;
        ++r;
        if (t + 1 < K) housekeeping<4 * G>(acc, f, r, c.fold_every, c.reduce_every, c);
        x0 = x0n;
        x1 = x1n;
#pragma unroll
        for (int g = 0; g < G; g++) p[g] = pn[g];
    }
#pragma unroll
    for (int g = 0; g < G; g++) {
        if ((u32)g < tile.count) {
            const u32 o = tile.out0 + g;
            const u64 bv = bias != nullptr ? bias[(size_t)o * limbs + limb] : 0;
            u64x2 v0, v1;
            v0.x = add_mod(acc_reduce(acc[4 * g + 0], c), bv, c.q);
            v0.y = add_mod(acc_reduce(acc[4 * g + 1], c), bv, c.q);
            v1.x = acc_reduce(acc[4 * g + 2], c);
            v1.y = acc_reduce(acc[4 * g + 3], c);
            u64* dst = out + ((size_t)o * 2 * limbs + limb) * N + n;
            if (accumulate & MAC_ACCUMULATE) {
                const u64x2 o0 = *reinterpret_cast<const u64x2*>(dst), o1 = *reinterpret_cast<const u64x2*>(dst + comp_stride);
                v0.x = add_mod(v0.x, o0.x, c.q);
                v0.y = add_mod(v0.y, o0.y, c.q);
                v1.x = add_mod(v1.x, o1.x, c.q);
                v1.y = add_mod(v1.y, o1.y, c.q);
            }
            *reinterpret_cast<u64x2*>(dst) = v0;
            *reinterpret_cast<u64x2*>(dst + comp_stride) = v1;
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

}  // namespace

// outputs that share their inputs with no other: gather their weights, then the streaming kernel
static int launch_scalar_single(he_ctx* ctx, const he_plan* plan, const ScalarSlice& sl, u32 limbs, const u64* ct_in, const u64* pt,
                                const u64* bias, u64* out, u64* wtab, u32 accumulate, hipStream_t s) {
    const u32 begin = sl.begin[0], count = sl.end[0] - begin;
    if (count == 0) return HE_OK;
    const Tile* tiles = plan->tiles_s_dev;
    const u32 n_tables = plan->table_s[sl.end[0] - 1] + 1 - sl.table_begin;
    hipLaunchKernelGGL(gather_weights_kernel, dim3(n_tables * GATHER_BLOCKS), dim3(256), 0, s, ctx->limbs, tiles, plan->wbase_s_dev,
                       plan->owners_dev + sl.table_begin, n_tables, limbs, plan->off_dev, plan->term_pt_dev, pt, wtab, sl.tab_words, sl.tab_skip,
                       sl.t_begin, sl.t_end);
    HE_HIP(hipGetLastError());
    const u32 per_thread = ctx->N >= 2048 ? 4 : 2;
    const u64 blocks = (u64)count * limbs * 2 * (ctx->N / (MAC_THREADS * 2 * per_thread));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((u32)blocks), dim3(MAC_THREADS), 0, s, ctx->limbs, limbs, ctx->N, tiles + begin, count, plan->wbase_s_dev + begin,
                           plan->term_ct_dev, wtab, sl.tab_words, sl.tab_skip, sl.t_begin, sl.t_end, ct_in, bias, out, accumulate);
    };
    auto launch_form = [&](auto stream) {
        constexpr bool STREAM = decltype(stream)::value;
        if (per_thread == 2) launch(mac_scalar_single_kernel<2, 8, STREAM>);
        else if (plan->max_terms_s[0] <= 2) launch(mac_scalar_single_kernel<4, 4, STREAM>);
        else launch(mac_scalar_single_kernel<4, 5, STREAM>);
    };
    if (mac_singles_stream(plan, limbs, ctx->N, accumulate & MAC_FOR_RESCALE)) launch_form(std::true_type{});
    else launch_form(std::false_type{});
    HE_HIP(hipGetLastError());
    return HE_OK;
}

static int launch_scalar_slice(he_ctx* ctx, const he_plan* plan, const ScalarSlice& sl, u32 limbs, const u64* ct_in, const u64* pt,
                               const u64* bias, u64* out, u64* wtab, u32 mode, hipStream_t s) {
    if (int rc = launch_scalar_single(ctx, plan, sl, limbs, ct_in, pt, bias, out, wtab, mode, s)) return rc;
    return launch_mac_digits(ctx, plan, sl, limbs, ct_in, pt, bias, out, wtab, mode, s);
}

// Terms [0, n_terms) of a slice in passes of `per_pass` (a multiple of 16): the first writes the canonical sums, the
// others add theirs (HE_ACCUMULATE).
static int launch_scalar_passes(he_ctx* ctx, const he_plan* plan, ScalarSlice& sl, u32 n_terms, u32 per_pass, u32 limbs, const u64* ct_in,
                                const u64* pt, const u64* bias, u64* out, u64* wtab, u32 mode, hipStream_t s) {
    for (u64 t = 0; t == 0 || t < n_terms; t += per_pass) {
        sl.t_begin = (u32)t;
        sl.t_end = (u32)std::min<u64>(t + per_pass, ~0u);
        const u32 pass_mode = n_terms <= per_pass ? mode : t == 0 ? mode & ~(u32)MAC_FOR_RESCALE : (u32)MAC_ACCUMULATE;
        if (int rc = launch_scalar_slice(ctx, plan, sl, limbs, ct_in, pt, t == 0 ? bias : nullptr, out, wtab, pass_mode, s)) return rc;
    }
    return HE_OK;
}

// The whole plan at once where its tables fit `wtab_bytes`, else range after range of tiles whose tables do, and a
// single table that does not in passes over its terms.  The matrix cores' 32-bit sums take DIGIT_MAX_TERMS terms.
static int launch_scalar(he_ctx* ctx, const he_plan* plan, u32 limbs, const u64* ct_in, const u64* pt, const u64* bias, u64* out, u64* wtab,
                         size_t wtab_bytes, u32 mode, hipStream_t s) {
    ScalarSlice sl;
    if (scalar_table_bytes(plan, limbs) <= wtab_bytes) {
        for (u32 cls = 0; cls < SCALAR_CLASSES; cls++) {
            sl.begin[cls] = plan->class_begin_s[cls];
            sl.end[cls] = plan->class_begin_s[cls + 1];
        }
        sl.table_begin = 0;
        sl.table_end = (u32)plan->table_end.size();
        sl.tab_skip = 0;
        sl.tab_words = plan->wtab_elems;
        return launch_scalar_passes(ctx, plan, sl, plan->max_terms, DIGIT_MAX_TERMS, limbs, ct_in, pt, bias, out, wtab, mode, s);
    }
    if (wtab_bytes < min_scalar_table_bytes(limbs)) return HE_ERR_WORKSPACE;
    const u64 room = wtab_bytes / sizeof(u64) / limbs / 4 * 4;  // words per limb
    for (u32 cls = 0; cls < SCALAR_CLASSES; cls++) {
        for (u32 i = plan->class_begin_s[cls]; i < plan->class_begin_s[cls + 1];) {
            for (u32 k = 0; k < SCALAR_CLASSES; k++) sl.begin[k] = sl.end[k] = 0;
            const u64 skip = plan->wbase_s[i];
            u32 end = i, n_terms = 0, per_pass = DIGIT_MAX_TERMS;
            while (end < plan->class_begin_s[cls + 1] && plan->table_end[plan->table_s[end]] - skip <= room)
                n_terms = std::max(n_terms, plan->tiles_s[end++].n_terms);
            if (end == i) {  // one table alone does not fit: all tiles that use it, in passes over their terms
                while (end < plan->class_begin_s[cls + 1] && plan->table_s[end] == plan->table_s[i]) end++;
                n_terms = plan->tiles_s[i].n_terms;
                const u64 words_per_16 = cls == 0 ? 16 : 512 * output_tiles(plan->tiles_s[i].count);
                per_pass = (u32)std::min<u64>(room / words_per_16 * 16, DIGIT_MAX_TERMS);
            }
            sl.begin[cls] = i;
            sl.end[cls] = end;
            sl.table_begin = plan->table_s[i];
            sl.table_end = plan->table_s[end - 1] + 1;
            sl.tab_skip = skip;
            sl.tab_words = room;
            if (int rc = launch_scalar_passes(ctx, plan, sl, n_terms, per_pass, limbs, ct_in, pt, bias, out, wtab, mode, s)) return rc;
            i = end;
        }
    }
    return HE_OK;
}

template <int G>
static int launch_poly_class(he_ctx* ctx, const he_plan* plan, int cls, u32 limbs, const u64* ct_in, const u64* pt,
                             const u64* bias, u64* out, u32 accumulate, hipStream_t s) {
    const u32 begin = plan->class_begin_p[cls], count = plan->class_begin_p[cls + 1] - begin;
    if (count == 0) return HE_OK;
    const u64 blocks = (u64)count * limbs * (ctx->N / (2 * MAC_THREADS));
    if (blocks > 0x7FFFFFFFull) return HE_ERR_RANGE;
    hipLaunchKernelGGL((mac_poly_kernel<G>), dim3((u32)blocks), dim3(MAC_THREADS), 0, s, ctx->limbs, limbs, ctx->N,
                       plan->tiles_p_dev + begin, count, plan->off_dev, plan->term_ct_dev, plan->term_pt_dev, pt, ct_in, bias, out, accumulate);
    HE_HIP(hipGetLastError());
    return HE_OK;
}

// The grid sizes launch_mac would use, checked without launching anything (the entry point calls this first,
// so that a plan too large for a grid is refused before any kernel of the call is on the stream).
int check_mac_launch(he_ctx* ctx, const he_plan* plan, u32 limbs, int pt_kind) {
    if (pt_kind == HE_PT_SCALAR) {
        const u64 singles = plan->class_begin_s[1] - plan->class_begin_s[0];
        const u32 per_thread = ctx->N >= 2048 ? 4 : 2;
        if (singles * limbs * 2 * (ctx->N / (MAC_THREADS * 2 * per_thread)) > 0x7FFFFFFFull) return HE_ERR_RANGE;
        if (singles * GATHER_BLOCKS > 0x7FFFFFFFull || mac_digits_blocks(ctx, plan, limbs) > 0x7FFFFFFFull) return HE_ERR_RANGE;
    } else {
        for (int cls = 0; cls < 3; cls++) {
            const u64 count = plan->class_begin_p[cls + 1] - plan->class_begin_p[cls];
            if (count * limbs * (ctx->N / (2 * MAC_THREADS)) > 0x7FFFFFFFull) return HE_ERR_RANGE;
        }
    }
    return HE_OK;
}

int launch_mac(he_ctx* ctx, const he_plan* plan, u32 limbs, const u64* ct_in, const u64* pt, int pt_kind, const u64* bias,
               u64* out, u64* wtab, size_t wtab_bytes, u32 accumulate, hipStream_t s) {
    int rc;
    if (pt_kind == HE_PT_SCALAR) {
        return launch_scalar(ctx, plan, limbs, ct_in, pt, bias, out, wtab, wtab_bytes, accumulate, s);
    } else {
        if ((rc = launch_poly_class<1>(ctx, plan, 0, limbs, ct_in, pt, bias, out, accumulate, s)) != HE_OK) return rc;
        if ((rc = launch_poly_class<2>(ctx, plan, 1, limbs, ct_in, pt, bias, out, accumulate, s)) != HE_OK) return rc;
        if ((rc = launch_poly_class<4>(ctx, plan, 2, limbs, ct_in, pt, bias, out, accumulate, s)) != HE_OK) return rc;
    }
    return HE_OK;
}
