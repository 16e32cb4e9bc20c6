// Ciphertext x scalar-plaintext multiply-accumulate (Alg. 8 summed over a plan) on the int8 matrix cores: groups of 2
// to 16 outputs that read the same ciphertexts (a dense layer's outputs, the filters of a convolution window).
//
// The arithmetic (he_arith.h, DigitConst): a residue is eight balanced base-256 digits, a term is a contraction of
// length 8 with eight int8 sums per output.  v_mfma_i32_32x32x32_i8 therefore takes FOUR terms (4 x 8 digits of the
// contraction) times FOUR outputs (4 x 8 sums) times 32 slots, and both operands are laid out by nature:
//  - the input operand of a lane is 16 consecutive contraction elements of one column: the residues of two terms at
//    one slot, as they lie in memory (their digits: one addition and an exclusive or per residue);
//  - of a result tile a lane holds 16 rows of one column; the table's rows are ordered so that those are the eight
//    sums of two outputs, and the final reduction of an output needs nothing from another lane.
// Residues in packed 32-bit storage (moduli below 2^30) have four digits and four sums: an instruction takes eight terms
// times eight outputs, the rest is the same.
//
// A term costs 64 int8 multiply-adds (2048 terms per compute unit and 32 cycles) instead of three or four 32-bit ones on
// the vector ALU, which only splits digits, forms addresses and reduces, about 25 instructions per output at the end.
// What bounds it: long sums, the inputs' way through the L2 (a dense layer's groups of 16 outputs each read all of
// them); a convolution window's 27 terms, the memory itself.  Measured against the same loop on 32-bit multiply-adds
// (the layer's MAC launch alone): dense 845 -> 100 at N = 2^13, L = 4: 1150 -> 345 us; dense 96 -> 24 at 2^15, L = 8:
// 358 -> 147 us; convolution 32x32x3, 3x3x16, at 2^14, L = 8: 5940 -> 3590 us (16 GB: 4.5 TB/s); 28x28, 5x5x5, at 2^13,
// L = 4: 435 -> 255 us; dense 64 -> 16 at 2^12, L = 2: 37 -> 13 us.  Packed, dense 1024 -> 256 at 2^12, L = 2: 352 -> 83 us.
// (On random digits the chip sustains 2.8 to 3.2 int8 POP/s, on constant ones 4.3: a long sum's arithmetic is priced with
// the former, 235 us of the 330 that 845 -> 96 takes; what else it waits for is the inputs, 75 us, and the meetings of
// the wavefronts around the table's stages, 35 us.)
// Tried: conditional loads at the ends of groups (the compiler's waits then drain the pipeline: 6200 us for the 2^14
// convolution); registers above the limit for two wavefronts per SIMD, whose reloads drain it as well (4500 us).
#include <algorithm>
#include <type_traits>

#include "he_internal.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef v4i v4i_mem __attribute__((aligned(8)));  // ... in the workspace (see u32x4)
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr u32 THREADS = 256, WAVES = THREADS / 64;
constexpr u32 CHUNK_TERMS = LIST_CHUNK;                     // terms that are in flight together (a chunk)
constexpr u32 RESIDENT_CHUNKS = 4;                          // tables of up to so many chunks stay in the LDS as a whole
constexpr u32 GROUPS_PER_WG = 16;                           // groups a workgroup runs through, at most
constexpr u64 MIN_WORKGROUPS = 2048;                        // ... while the launch keeps at least this many workgroups
static_assert(DIGIT_MAX_TERMS % CHUNK_TERMS == 0, "the parts of a long sum are whole chunks");
static_assert(BLOCK_TERMS == 32 / sizeof(u64), "the terms that one instruction contracts");

// What the storage form of a residue sets (V = u64 or u32): its digits D fill sizeof(V) bytes of the contraction, an
// output has D sums.
template <typename V>
struct Form {
    static constexpr u32 D = sizeof(V);
    static constexpr u32 BLOCK_TERMS = 32 / D;              // terms of one matrix instruction
    static constexpr u32 LANE_TERMS = 16 / D;               // ... of which a lane holds so many
    static constexpr u32 CHUNK_BLOCKS = CHUNK_TERMS / BLOCK_TERMS;
    static constexpr u32 TILE_OUTPUTS = 32 / D;             // outputs of one result tile
    static constexpr u32 LANE_OUTPUTS = 16 / D;             // ... of which a lane holds so many
    static constexpr int CT = 16 / D;                       // column tiles (of 32 slots) of a wavefront: a lane's 16 bytes of a row
    static constexpr u32 SLOTS = WAVES * 32 * CT;           // slots of a workgroup
    __host__ __device__ static constexpr u32 tiles(u32 count) { return D == 8 ? output_tiles(count) : count <= 8 ? 1 : 2; }
};

template <typename T>
__device__ __forceinline__ T uniform_load(const T* p) {  // read-only, workgroup-uniform data: a scalar load
    return *(const __attribute__((address_space(4))) T*)(p);
}

// Workgroup barrier that orders LDS traffic only (a full __syncthreads() would also wait for the inputs that are
// deliberately in flight).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ---------------------------------------------------------------------------------------------
// The table: for every distinct group of plaintexts and every limb, tiles [block of terms][outputs] of 64 lanes x 16 bytes,
// the matrix instruction's operand as the lanes read it.  Lane (row r, half h) holds row r's elements of half h's terms of
// the block: positions h * LANE_TERMS .. of the order in which the term lists are stored (he_plan::lists_dev).  Row r
// belongs to half (r >> 2) & 1 of the tile's outputs and there to sum (r & 3) + 4 * (r >> 3) of the 16 of that half's lanes.
// Terms beyond the group's (up to a multiple of `pad`: whole chunks, or one block for a plan of short sums, see SHORT) and
// outputs beyond its count are zeros.  One thread: one (term, output) of limb blockIdx.z and table blockIdx.y; the lanes that fill
// a tile between them are neighbours, the terms of one 16-byte operand next to one another.  (With the limbs fastest every
// store went to a line of its own: layer 500 -> 256 at 2^12, L = 8 619 -> 601 us, packed 1024 -> 256 101 -> 97.)
template <typename V>
__global__ void __launch_bounds__(256) gather_digits_kernel(DigitTable dt, const Tile* tiles, const u64* wbase, const u32* owners, u32 limbs,
                                                            const u32* off, const u32* term_pt, const u64* pt, u64* tab, u64 tab_words,
                                                            u64 tab_skip, u32 t_begin, u32 t_end, u32 pad) {
    using F = Form<V>;
    constexpr u32 LANE_TERMS = F::LANE_TERMS, TILE_OUTPUTS = F::TILE_OUTPUTS;
    const u32 tile_i = uniform_load(owners + blockIdx.y), limb = blockIdx.z;
    const Tile tile = tiles[tile_i];
    const u32 first = min(t_begin, tile.n_terms), K = min(t_end, tile.n_terms) - first;
    const u32 ot = F::tiles(tile.count);  // 1, 2 or 4
    const u32 total = (K + pad - 1) / pad * pad * ot * TILE_OUTPUTS;
    const DigitConst& c = dt.c[limb];
    V* dst = reinterpret_cast<V*>(tab + (wbase[tile_i] - tab_skip) + (u64)limb * tab_words);
    for (u32 i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        // which element of a lane's operand, which half, which of the tile's outputs, which tile of which block
        const u32 j = i % LANE_TERMS, half = i / LANE_TERMS % 2, oo = i / (2 * LANE_TERMS) % TILE_OUTPUTS;
        const u32 at_tile = i / (2 * LANE_TERMS * TILE_OUTPUTS);
        const u32 o = at_tile % ot * TILE_OUTPUTS + oo, block = at_tile / ot;
        // position `at` of the half's part of its chunk's list order [half][block of 4][2]
        const u32 at = block % F::CHUNK_BLOCKS * LANE_TERMS + j;
        const u32 t = block / F::CHUNK_BLOCKS * CHUNK_TERMS + (at >> 1) * 4 + half * 2 + (at & 1);
        V row[F::D] = {};
        if (o < tile.count && t < K) plaintext_digits(pt[(size_t)term_pt[off[tile.out0 + o] + first + t] * limbs + limb], c, row);
        V* out = dst + ((size_t)at_tile * 64 + 32 * half) * LANE_TERMS + j;
#pragma unroll
        for (u32 m = 0; m < F::D; m++) {
            const u32 k = oo % F::LANE_OUTPUTS * F::D + m;  // which of the lane's 16 sums
            out[((k & 3) + 8 * (k >> 2) + 4 * (oo / F::LANE_OUTPUTS)) * LANE_TERMS] = row[m];
        }
    }
}

// ---------------------------------------------------------------------------------------------
template <typename V>
struct MacArgs {
    const DigitTile* tiles;
    const u32* lists;
    const u64* tab;         // gathered tables
    u64 tab_words;          // words per limb
    u64 tab_skip;           // where the tables in `tab` start in the plan's numbering
    const V* ct_in;
    const u64* bias;
    V* out;
    u32 limbs, N;
    u32 t_begin, t_end;     // the range of every group's terms to take, multiples of 16 (all of them: 0, 2^32 - 1)
    u32 mode;               // MAC_* bits
};

__device__ __forceinline__ DigitTile load_tile(const DigitTile* p) {  // 32 bytes, one scalar load
    typedef u32 u32x8 __attribute__((ext_vector_type(8)));
    const u32x8 v = *(const __attribute__((address_space(4))) u32x8*)(p);
    return DigitTile{v[0], v[1], v[2], v[3], ((u64)v[5] << 32) | v[4], v[6], v[7]};
}

// Where a wavefront is in its stream of chunks.
struct Cursor {
    u32 tile, chunk, n_chunks;
    u32 list;             // the group's term list, in chunks
    u32 piece;            // the group's table, in 16-byte pieces from the limb's part
};

template <typename V>
__device__ __forceinline__ u32 chunks_of(const MacArgs<V>& a, const DigitTile& t) {
    const u32 K = min(a.t_end, t.n_terms) - min(a.t_begin, t.n_terms);
    return __builtin_amdgcn_readfirstlane((K + CHUNK_TERMS - 1) / CHUNK_TERMS);
}

template <typename V>
__device__ __forceinline__ void enter_group(Cursor& p, const MacArgs<V>& a, u32 tile) {
    const DigitTile t = load_tile(a.tiles + tile);
    const u32 first = min(a.t_begin, t.n_terms);
    // (readfirstlane: the cursor stays in scalar registers)
    p.tile = __builtin_amdgcn_readfirstlane(tile);
    p.chunk = 0;
    p.n_chunks = chunks_of(a, t);
    p.list = __builtin_amdgcn_readfirstlane(t.list + first / CHUNK_TERMS);
    p.piece = __builtin_amdgcn_readfirstlane((u32)((t.words - a.tab_skip) / 2));
}

// The chunk after this one; after the last one of the stream the cursor stays (its loads are repeated, never used).
template <typename V>
__device__ __forceinline__ void step(Cursor& p, const MacArgs<V>& a, u32 tile_end, u32 stride) {
    if (p.chunk + 1 < p.n_chunks) p.chunk = __builtin_amdgcn_readfirstlane(p.chunk + 1);
    else if (p.tile + stride < tile_end) enter_group(p, a, p.tile + stride);
}

// A wavefront's share of a group of outputs: OT x CT result tiles.  Column tile k holds slot k of the lanes' CT adjacent
// slots.
template <typename V, int OT>
struct Sums {
    static constexpr int CT = Form<V>::CT;
    static constexpr u32 D = Form<V>::D;
    v16i t[OT][CT];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int o = 0; o < OT; o++)
#pragma unroll
            for (int k = 0; k < CT; k++)
#pragma unroll
                for (int i = 0; i < 16; i++) t[o][k][i] = 0;
    }
    // the sums of this lane's output i of tile o at its slot k
    __device__ __forceinline__ void get(int32_t (&r)[D], int o, int k, int i) const {
#pragma unroll
        for (u32 m = 0; m < D; m++) r[m] = t[o][k][i * D + m];
    }
};

// What a workgroup works on: one slice of one (component, limb) row.
template <typename V>
struct Slice {
    u32 comp, limb, lane, half;
    u32 ct_stride;       // bytes (below 2^32 for 16 limbs of 2^15 residues)
    const char* x_base;  // this lane's slots of ciphertext 0
    const v4i_mem* tab;  // the limb's tables
    V* dst;              // this lane's slots of output 0
};

// Final reduction, bias (Alg. 4) and store of one group.  The caller has waited for its loads in flight: a later wait
// for one of them would wait for these stores as well.
// STREAM: the stores go past the caches (mac_groups_stream), an instance of its own of every kernel.  Chosen by a branch per output
// instead, both kinds were slower: dense 64 -> 16 at N = 2^12 16.5 us, 16.2 now; packed, 512 outputs of 16 terms in groups of 16 at 2^13 28.2
// and 27.4; past the caches 4096 outputs of one term in groups of 16, N = 2^13, L = 4, 564 and 538.
template <typename V, int OT, bool STREAM>
__device__ __forceinline__ void store_group(const Sums<V, OT>& sums, const MacArgs<V>& a, const Slice<V>& w, const DigitConst& c, u32 out0, u32 count) {
    using F = Form<V>;
    constexpr u32 LANE_OUTPUTS = F::LANE_OUTPUTS, TILE_OUTPUTS = F::TILE_OUTPUTS, D = F::D;
    constexpr int CT = F::CT;
    const size_t out_stride = (size_t)2 * a.limbs * a.N;
    u32 half = w.half;
    asm volatile("" : "+v"(half));  // what follows is derived here, not kept in registers through the loop over terms
    V* dst = w.dst + (size_t)out0 * out_stride + half * (LANE_OUTPUTS * out_stride);
    const u32 lazy = D == 8 && (a.mode & MAC_FOR_RESCALE) && w.limb + 1 < a.limbs ? c.lazy : 0;
    const bool accumulate = a.mode & MAC_ACCUMULATE;
    // The bias residues come in with scalar loads, those of the next four outputs while four are reduced.  (Without a
    // bias the loads read the group's descriptor and are masked.)
    const bool has_bias = a.bias != nullptr && w.comp == 0;
    const char* bias0 = has_bias ? reinterpret_cast<const char*>(a.bias + (size_t)out0 * a.limbs + w.limb) : reinterpret_cast<const char*>(a.tiles);
    const u32 bias_step = has_bias ? a.limbs * 8 : 0;
    const u64 mask = has_bias ? ~0ull : 0;
    // step s handles outputs s * 2 .. of both halves
    constexpr int STEPS = OT * LANE_OUTPUTS / 2;
    auto output_of = [&](int s, int i, u32 h) -> u32 {  // output i (0, 1) of step s in half h
        return (u32)(s * 2 / LANE_OUTPUTS) * TILE_OUTPUTS + h * LANE_OUTPUTS + (u32)(s * 2 % LANE_OUTPUTS) + i;
    };
    auto load_bias = [&](u64 (&b)[4], int s) {
#pragma unroll
        for (u32 g = 0; g < 4; g++) b[g] = uniform_load(reinterpret_cast<const u64*>(bias0 + min(output_of(s, g & 1, g >> 1), count - 1) * bias_step));
    };
    auto reduce_all = [&](auto reduce) {
        u64 next[4];
        load_bias(next, 0);
#pragma unroll
        for (int s = 0; s < STEPS; s++) {
            u64 start[4];  // [half][i]
#pragma unroll
            for (int g = 0; g < 4; g++) {
                start[g] = D == 8 ? c.start + (next[g] & mask) : add_mod(c.start, next[g] & mask, c.q);
                asm volatile("" : "+s"(start[g]));
            }
            if (s + 1 < STEPS) load_bias(next, s + 1);
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const u64 st = half ? start[2 + i] : start[i];
                const bool mine = output_of(s, i, half) < count;
                V* const at = dst + output_of(s, i, 0) * out_stride;
                V v[CT];
#pragma unroll
                for (int k = 0; k < CT; k++) {
                    int32_t r[D];
                    sums.get(r, s * 2 / LANE_OUTPUTS, k, s * 2 % LANE_OUTPUTS + i);
                    v[k] = reduce(r, st);
                }
                if (mine) {
                    typedef V row_piece __attribute__((ext_vector_type(CT), aligned(8)));  // 16 bytes (see u64x2)
                    if (accumulate) {
                        const row_piece old = *reinterpret_cast<const row_piece*>(at);
#pragma unroll
                        for (int k = 0; k < CT; k++) v[k] = add_mod(v[k], old[k], c.q);
                    }
                    row_piece all;
#pragma unroll
                    for (int k = 0; k < CT; k++) all[k] = v[k];
                    if constexpr (STREAM) __builtin_nontemporal_store(all, reinterpret_cast<row_piece*>(at));
                    else *reinterpret_cast<row_piece*>(at) = all;
                }
                __builtin_amdgcn_sched_barrier(0);  // one output at a time: its temporaries are few
            }
        }
    };
    if constexpr (D == 8) {  // (one uniform branch for the whole group)
        if (lazy == 1) reduce_all([&](const int32_t (&r)[8], u64 st) { return digit_reduce_lazy(r, st, c); });
        else if (lazy == 2) reduce_all([&](const int32_t (&r)[8], u64 st) { return digit_reduce_lazy4(r, st, c); });
        else reduce_all([&](const int32_t (&r)[8], u64 st) { return digit_reduce(r, st, c); });
    } else {
        reduce_all([&](const int32_t (&r)[4], u64 st) { return digit_reduce32(r, (u32)st, c); });
    }
}

// the balanced digits of two residues, given as 32-bit words
__device__ __forceinline__ v4i digits_of(u32 a0, u32 a1, u32 b0, u32 b1) {
    const u64 a = balanced_digits(((u64)a1 << 32) | a0), b = balanced_digits(((u64)b1 << 32) | b0);
    return v4i{(int)(u32)a, (int)(u32)(a >> 32), (int)(u32)b, (int)(u32)(b >> 32)};
}

// A block's matrix operand for column tile k from the lane's residues of its LANE_TERMS terms
__device__ __forceinline__ v4i operand(const u32x4 (&x)[2], int k) { return digits_of(x[0][2 * k], x[0][2 * k + 1], x[1][2 * k], x[1][2 * k + 1]); }
__device__ __forceinline__ v4i operand(const u32x4 (&x)[4], int k) {
    return v4i{(int)balanced_digits32(x[0][k]), (int)balanced_digits32(x[1][k]), (int)balanced_digits32(x[2][k]), (int)balanced_digits32(x[3][k])};
}

// Every `stride`-th of the groups tile_first .. tile_end - 1 as one stream of chunks (16 terms each, the last of a group padded with zero
// weights).  A wavefront multiplies the inputs it requested a chunk ago, requests those of the next chunk, also across
// the end of a group, and the term list of the chunk after that; all of it is straight-line code, so that a wait is
// for the loads it needs and no others.
// RESIDENT: the groups share one table, which the workgroup has put into the LDS; the wavefronts do not meet.
// Otherwise the workgroup brings the next chunk's table tiles into the other half of the LDS meanwhile.
// SHORT: no group of the plan has more terms than one block takes (1x1 convolutions over few channels), and a chunk is that
// one block: with the other three as padding a quarter of the loads and products were of use.  (N = 2^13, L = 4: 256 groups of
// 16 outputs and one term with plaintexts of their own 1000 -> 785 us, 935 on the vector ALU; of two outputs that share their
// plaintexts 197 -> 135.)
template <typename V, int OT, bool RESIDENT, bool SHORT, bool STREAM>
__device__ __forceinline__ void mac_stream(const MacArgs<V>& a, const Slice<V>& w, const DigitConst& c, u32 tile_first, u32 tile_end, u32 stride, v4i* lds) {
    using F = Form<V>;
    static_assert(!SHORT || (RESIDENT && F::LANE_TERMS <= 4), "one chunk, its list in one piece");
    constexpr u32 CHUNK_BLOCKS = SHORT ? 1 : F::CHUNK_BLOCKS, LANE_TERMS = F::LANE_TERMS;
    constexpr int CT = F::CT;
    constexpr u32 CHUNK_PIECES = CHUNK_BLOCKS * OT * 64;  // 16-byte pieces of a chunk's tiles
    constexpr u32 PER_THREAD = CHUNK_PIECES < THREADS ? 1 : CHUNK_PIECES / THREADS;
    static_assert(CHUNK_PIECES % THREADS == 0 || THREADS % CHUNK_PIECES == 0, "every thread brings the same number of pieces");
    Cursor cur, nxt, after;
    enter_group(cur, a, tile_first);
    nxt = cur;
    step(nxt, a, tile_end, stride);
    after = nxt;
    step(after, a, tile_end, stride);

    u32 idx[8];                            // ciphertexts of the eight terms that this lane reads in the next chunk
    u32x4 x[CHUNK_BLOCKS][LANE_TERMS];     // residues of this chunk, 16 bytes of a row each
    auto request_idx = [&](const Cursor& p, u32 part) {  // four at a time: 16 bytes
        const u32x4 v = *reinterpret_cast<const u32x4*>(a.lists + (size_t)(p.list + p.chunk) * LIST_CHUNK + (8 * w.half + 4 * part));
#pragma unroll
        for (u32 k = 0; k < 4; k++) idx[4 * part + k] = v[k];
    };
    auto request_x = [&](u32 b) {
#pragma unroll
        for (u32 j = 0; j < LANE_TERMS; j++) x[b][j] = *reinterpret_cast<const u32x4*>(w.x_base + (u64)idx[b * LANE_TERMS + j] * w.ct_stride);
    };
    // (with fewer pieces than threads some pieces are brought twice)
    v4i stage[PER_THREAD];
    auto request_tiles = [&](const Cursor& p) {
        const v4i_mem* src = w.tab + (p.piece + (u64)p.chunk * CHUNK_PIECES);
#pragma unroll
        for (u32 i = 0; i < PER_THREAD; i++) stage[i] = src[(i * THREADS + threadIdx.x) % CHUNK_PIECES];
    };
    auto write_tiles = [&](u32 buf) {
#pragma unroll
        for (u32 i = 0; i < PER_THREAD; i++) lds[buf * CHUNK_PIECES + (i * THREADS + threadIdx.x) % CHUNK_PIECES] = stage[i];
    };
    u32 buf = 0;
    if constexpr (!RESIDENT) request_tiles(cur);
    request_idx(cur, 0);
    if constexpr (!SHORT) request_idx(cur, 1);
#pragma unroll
    for (u32 b = 0; b < CHUNK_BLOCKS; b++) request_x(b);
    request_idx(nxt, 0);
    if constexpr (!SHORT) request_idx(nxt, 1);
    if constexpr (!RESIDENT) write_tiles(0);
    while (true) {
        const u32 tile = cur.tile, chunks = cur.n_chunks;
        Sums<V, OT> sums;
        // FIRST: the first block's products start the sums
        auto run_chunk = [&](u32 chunk, auto first) {
            constexpr bool FIRST = decltype(first)::value;
            if constexpr (!RESIDENT) {
                lds_barrier();  // this chunk's tiles are in place, and nobody reads the other half any more
                request_tiles(nxt);
            }
            const v4i* tiles = lds + (RESIDENT ? chunk : buf) * CHUNK_PIECES + w.lane;
#pragma unroll
            for (u32 b = 0; b < CHUNK_BLOCKS; b++) {
                v4i in[CT];
#pragma unroll
                for (int k = 0; k < CT; k++) in[k] = operand(x[b], k);
                request_x(b);
                if (SHORT || (b + 1) * LANE_TERMS == 4) request_idx(after, 0);
                if ((b + 1) * LANE_TERMS == 8) request_idx(after, 1);
#pragma unroll
                for (int o = 0; o < OT; o++) {
                    const v4i t = tiles[(b * OT + o) * 64];
                    const v16i zero = {};
#pragma unroll
                    for (int k = 0; k < CT; k++)
                        sums.t[o][k] = __builtin_amdgcn_mfma_i32_32x32x32_i8(t, in[k], FIRST && b == 0 ? zero : sums.t[o][k], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!RESIDENT) write_tiles(buf ^ 1);
            buf ^= 1;
            nxt = after;
            step(after, a, tile_end, stride);
        };
        run_chunk(0, std::true_type{});
#pragma unroll 1
        for (u32 chunk = 1; chunk < chunks; chunk++) run_chunk(chunk, std::false_type{});
#pragma unroll
        for (u32 b = 0; b < CHUNK_BLOCKS; b++)
#pragma unroll
            for (u32 j = 0; j < LANE_TERMS; j++) asm volatile("" : "+v"(x[b][j]));  // the next chunk's inputs have arrived
        const DigitTile t = load_tile(a.tiles + tile);
        store_group<V, OT, STREAM>(sums, a, w, c, t.out0, t.count);
        if (tile + stride >= tile_end) break;
        cur.tile = tile + stride;
        cur.n_chunks = chunks_of(a, load_tile(a.tiles + tile + stride));
    }
}

// 16-byte pieces of table tiles that a workgroup keeps in its LDS
template <typename V, bool SHORT>
constexpr u32 lds_pieces(int ot) { return (SHORT ? 1 : RESIDENT_CHUNKS * Form<V>::CHUNK_BLOCKS) * ot * 64; }

struct MacClass {
    u32 first, end, per_wg, blocks;  // the class's groups among the plan's tiles, groups per workgroup and workgroups
    u32 runs;                        // ... workgroups per slice of a row
    u32 abreast;                     // 1: the wavefronts of a workgroup take neighbouring groups over one slice of 32 * CT slots,
                                     // 0: one group over a slice each
    template <typename V>
    __host__ __device__ u32 slots() const { return abreast ? Form<V>::SLOTS / WAVES : Form<V>::SLOTS; }
};

// Where a workgroup is: slice of the row fastest, then run of groups, then (component, limb): workgroups go to the eight XCDs
// round-robin and the number of slices is a multiple of eight from N = 2^11 on (packed residues: 2^12), so the same slice of neighbouring groups (which
// read the same or overlapping inputs) runs on the same XCD, close in time, and hits in its L2.
struct MacPlace {
    u32 part, run, row;  // row: (limb, component)
};
__device__ __forceinline__ MacPlace mac_place(u32 b, u32 parts, u32 runs, u32 first_row = 0) {
    const u32 rest = b / parts;
    return MacPlace{b % parts, rest % runs, first_row + rest / runs};
}

// MIXED: one of several classes of a launch, whose windows never go abreast.  (With the choice left open the three branches of that kernel
// had 146 scalar registers parked in vector lanes, 103 now: dense 300 -> 37 at N = 2^13, L = 2 32.8 -> 32.2 us, 300 -> 23 at L = 3
// 39.2 -> 38.6.  An opaque place in each branch parks 92 to 104 and was better for some launches, 845 -> 20 at L = 4 119 -> 110 to 116, and
// worse for others, 200 + 113 -> 37 in two calls 116.7 -> 118.4.)
template <typename V, int OT, bool SHORT, bool STREAM, bool MIXED = false>
__device__ __forceinline__ void mac_class(const MacPlace& at_wg, const MacArgs<V>& a, const DigitTable& dt, const MacClass& m, v4i* lds) {
    using F = Form<V>;
    const u32 part = at_wg.part;
    const bool abreast = !MIXED && !SHORT && sizeof(V) == sizeof(u64) && m.abreast;  // (go_abreast)
    const u32 tile_first = m.first + at_wg.run * m.per_wg;
    const u32 tile_end = min(tile_first + m.per_wg, m.end);
    Slice<V> w;
    w.comp = at_wg.row & 1;
    w.limb = at_wg.row >> 1;
    w.lane = threadIdx.x % 64;
    w.half = w.lane / 32;
    w.ct_stride = 2 * a.limbs * a.N * sizeof(V);
    const size_t at = ((size_t)w.comp * a.limbs + w.limb) * a.N + part * (abreast ? F::SLOTS / WAVES : F::SLOTS) + (abreast ? 0 : threadIdx.x / 64 * (32 * F::CT)) + F::CT * (w.lane % 32);
    w.x_base = reinterpret_cast<const char*>(a.ct_in + at);
    w.dst = a.out + at;
    w.tab = reinterpret_cast<const v4i_mem*>(a.tab + (u64)w.limb * a.tab_words);
    // the constants of the reduction, fetched once and held in scalar registers (left to itself the compiler fetches
    // them again for every output, and waits each time)
    DigitConst c = dt.c[w.limb];
    asm volatile("" : "+s"(c.q), "+s"(c.start), "+s"(c.hi_offset), "+s"(c.top), "+s"(c.mult), "+s"(c.mult_shift), "+s"(c.hi_shift), "+s"(c.kappa8), "+s"(c.lazy), "+s"(c.b8), "+s"(c.b16), "+s"(c.b24));
    for (u32 tile = tile_first; tile < tile_end;) {
        Cursor p;
        enter_group(p, a, tile);
        const DigitTile t = load_tile(a.tiles + tile);
        if (p.n_chunks == 0) {  // no terms: the bias alone
            Sums<V, OT> zero;
            zero.clear();
            store_group<V, OT, STREAM>(zero, a, w, c, t.out0, t.count);
            tile++;
        } else if (SHORT || p.n_chunks <= RESIDENT_CHUNKS) {
            const u32 end = min(tile_end, t.same_until);
            const u32 pieces = SHORT ? OT * 64 : p.n_chunks * F::CHUNK_BLOCKS * OT * 64;
            lds_barrier();  // (the table of the groups before is no longer read)
            for (u32 i = threadIdx.x; i < pieces; i += THREADS) lds[i] = w.tab[p.piece + i];
            lds_barrier();
            const u32 own = abreast ? tile + __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : tile;
            if (own < end) mac_stream<V, OT, true, SHORT, STREAM>(a, w, c, own, end, abreast ? WAVES : 1, lds);
            tile = end;
        } else {
            // the rest of the run: groups with long sums follow one another (tables of a class are in the order of
            // their first use, so a shorter one may still come and takes the same path)
            if constexpr (!SHORT) {
                lds_barrier();
                mac_stream<V, OT, false, false, STREAM>(a, w, c, tile, tile_end, 1, lds);
            }
            tile = tile_end;
        }
    }
}

// 64-bit residues: groups of 9..16 (OT = 4), 5..8 (2) and 2..4 (1) outputs; packed ones: of 9..16 (2) and up to 8 (1).
// The accumulators, OT x CT x 16 registers, set how many wavefronts a SIMD holds.
template <typename V, int OT, bool SHORT, bool STREAM>
__global__ void __launch_bounds__(THREADS, OT * Form<V>::CT == 8 ? 2 : OT * Form<V>::CT == 4 ? 3 : 4)
mac_digits_kernel(DigitTable dt, MacArgs<V> a, MacClass m) {
    __shared__ v4i lds[lds_pieces<V, SHORT>(OT)];
    const MacPlace at = mac_place(blockIdx.x, a.N / m.template slots<V>(), m.runs);
    mac_class<V, OT, SHORT, STREAM>(at, a, dt, m, lds);
}

// A plan with groups of several classes in one launch, all groups of one slice next to one another: they read the same inputs.
// (With the workgroups of the largest class first and the others behind them the inputs of a dense layer 96 -> 24 at 2^15, L = 8,
// came from the memory twice: 186 us, now 150; 845 -> 100 at 2^13, L = 8, 800 and 756.)  In the last `tail` rows, about as
// many workgroups as the chip holds, the largest class does come first and the smaller ones fill in while it drains.
template <typename V, bool SHORT, bool STREAM>
__global__ void __launch_bounds__(THREADS, 2) mac_digits_mixed_kernel(DigitTable dt, MacArgs<V> a, MacClass c16, MacClass c8, MacClass c4, u32 tail) {
    constexpr int OT16 = Form<V>::tiles(16), OT8 = Form<V>::tiles(8), OT4 = Form<V>::tiles(4);
    __shared__ v4i lds[lds_pieces<V, SHORT>(OT16)];
    const u32 parts = a.N / Form<V>::SLOTS, lead = a.limbs * 2 - tail, runs = c16.runs + c8.runs + c4.runs;
    u32 b = blockIdx.x, cls;
    MacPlace at;
    if (b < lead * parts * runs) {
        at = mac_place(b, parts, runs);
        cls = at.run < c16.runs ? 0 : at.run < c16.runs + c8.runs ? 1 : 2;
        at.run -= cls == 0 ? 0 : cls == 1 ? c16.runs : c16.runs + c8.runs;
    } else {
        b -= lead * parts * runs;
        const u32 n16 = tail * parts * c16.runs, n8 = tail * parts * c8.runs;
        cls = b < n16 ? 0 : b < n16 + n8 ? 1 : 2;
        at = mac_place(b - (cls == 0 ? 0 : cls == 1 ? n16 : n16 + n8), parts, cls == 0 ? c16.runs : cls == 1 ? c8.runs : c4.runs, lead);
    }
    if (cls == 0) mac_class<V, OT16, SHORT, STREAM, true>(at, a, dt, c16, lds);
    else if (cls == 1) mac_class<V, OT8, SHORT, STREAM, true>(at, a, dt, c8, lds);
    else mac_class<V, OT4, SHORT, STREAM, true>(at, a, dt, c4, lds);
}

// Groups per workgroup and workgroups of one class over the tiles [first, end).  Several groups per workgroup pay the
// start of a run (descriptor -> term list -> inputs, and a convolution's table) once; a group without terms stays alone.
// abreast: a convolution's windows that follow one another share most of their inputs.  With a window per wavefront, all over
// the same slots and in step, what one wavefront reads the next finds in the L1 (loads, not products, bind a convolution with
// few filters).  Such a workgroup covers a quarter of the slots and takes up to four times the groups.  Only where one table that
// stays in the LDS serves all groups (unpadded convolutions): 28x28x1, 5x5x5, N = 2^13, L = 4, 274 -> 254 us; 12x12x7, 3x3x16,
// L = 3 411 -> 392; 30x30x1, 5x5x12, 2^12, 898 and 904.  The runs of a padded one end with every table: 10x10x3, 3x3x5, 2^15
// 682 -> 755, 16x16x2, 3x3x4, 2^13 234 -> 256.
template <typename V>
MacClass mac_class_of(const he_ctx* ctx, const he_plan* plan, u32 limbs, u32 cls, u32 first, u32 end, u32 t_begin, bool abreast = false) {
    MacClass m{first, end, 1, 0, 0, abreast};
    const u64 per_run = (u64)limbs * 2 * (ctx->N / m.slots<V>());
    const u32 count = end - first, least = abreast ? WAVES : 1;
    m.per_wg = plan->min_terms_s[cls] > t_begin ? GROUPS_PER_WG * least : 1;  // (a stream has no group without terms in it)
    while (m.per_wg > least && (u64)((count + m.per_wg - 1) / m.per_wg) * per_run < MIN_WORKGROUPS) m.per_wg /= 2;
    m.runs = (count + m.per_wg - 1) / m.per_wg;
    if (abreast && m.runs) m.per_wg = (count + m.runs * WAVES - 1) / (m.runs * WAVES) * WAVES;  // runs of equal length
    m.blocks = (u32)std::min<u64>(m.runs * per_run, 0x7FFFFFFFull);
    return m;
}

// Whether the groups [first, end) of a class go abreast (mac_class_of) where they are all that a launch over `n_tables` tables has.
template <typename V>
bool go_abreast(const he_ctx* ctx, const he_plan* plan, u32 limbs, u32 cls, u32 first, u32 end, u32 t_begin, u32 n_tables, MacClass& m) {
    if (sizeof(V) != sizeof(u64) || !plan->shared_inputs_s[cls] || plan->short_sums() || plan->min_terms_s[cls] <= t_begin ||
        plan->max_terms_s[cls] > RESIDENT_CHUNKS * CHUNK_TERMS || n_tables != 1 || end - first < 2 * WAVES)
        return false;
    const MacClass abreast = mac_class_of<V>(ctx, plan, limbs, cls, first, end, t_begin, true);
    if (abreast.blocks >= 0x7FFFFFFFu) return false;
    m = abreast;
    return true;
}

template <typename V, bool SHORT, bool STREAM>
void launch_classes(he_ctx* ctx, const MacArgs<V>& a, const MacClass (&c)[SCALAR_CLASSES], u64 blocks, hipStream_t s) {
    const dim3 grid((u32)blocks), block(THREADS);
    constexpr int OT16 = Form<V>::tiles(16), OT8 = Form<V>::tiles(8), OT4 = Form<V>::tiles(4);
    if (c[3].blocks == blocks) hipLaunchKernelGGL((mac_digits_kernel<V, OT16, SHORT, STREAM>), grid, block, 0, s, ctx->digits, a, c[3]);
    else if (c[2].blocks == blocks) hipLaunchKernelGGL((mac_digits_kernel<V, OT8, SHORT, STREAM>), grid, block, 0, s, ctx->digits, a, c[2]);
    else if (c[1].blocks == blocks) hipLaunchKernelGGL((mac_digits_kernel<V, OT4, SHORT, STREAM>), grid, block, 0, s, ctx->digits, a, c[1]);
    else {
        const u32 rows = a.limbs * 2;
        const u64 resident = 2 * 256;  // two workgroups per compute unit
        // (Less than two waves of workgroups of which the largest class is four fifths or more are all tail: N = 2^13, L = 3, 300 -> 68,
        // four runs of groups of 16 and one of 4, 76.7 us, 79.2 with a row in the order of the rows; 300 -> 100 at L = 2 65.0 and 66.5.
        // Where the classes are closer to one another what they share counts for more: 500 -> 24 at 2^14, L = 3 146 us and 125;
        // 200 -> 40 at 2^12, L = 8 54.4 and 50.4.)
        const bool all_tail = blocks < 2 * resident && 4 * (c[2].runs + c[1].runs) <= c[3].runs;
        const u32 tail = all_tail ? rows : (u32)std::min<u64>(rows, (resident * rows + blocks - 1) / blocks);
        hipLaunchKernelGGL((mac_digits_mixed_kernel<V, SHORT, STREAM>), grid, block, 0, s, ctx->digits, a, c[3], c[2], c[1], tail);
    }
}

template <typename V>
int launch_mac_digits_t(he_ctx* ctx, const he_plan* plan, const ScalarSlice& sl, u32 limbs, const V* ct_in, const u64* pt, const u64* bias, V* out,
                        u64* wtab, u32 mode, hipStream_t s) {
    MacClass c[SCALAR_CLASSES];
    u64 blocks = 0;
    u32 first = ~0u;  // the first tile of the slice in these classes
    for (u32 cls = 1; cls < SCALAR_CLASSES; cls++) {
        c[cls] = mac_class_of<V>(ctx, plan, limbs, cls, sl.begin[cls], sl.end[cls], sl.t_begin);
        blocks += c[cls].blocks;
        if (sl.begin[cls] < sl.end[cls]) first = std::min(first, sl.begin[cls]);
    }
    if (blocks == 0) return HE_OK;
    const u32 table0 = plan->table_s[first];
    for (u32 cls = 1; cls < SCALAR_CLASSES; cls++) {
        if (c[cls].blocks == blocks && go_abreast<V>(ctx, plan, limbs, cls, sl.begin[cls], sl.end[cls], sl.t_begin, sl.table_end - table0, c[cls]))
            blocks = c[cls].blocks;
    }
    const bool short_sums = sizeof(V) == sizeof(u64) && plan->short_sums();  // (packed sums that short run on the vector ALU)
    // about one entry per thread, but no more workgroups than fill the chip a few times
    const u64 entries = (u64)std::min(plan->max_terms, sl.t_end - sl.t_begin) * 16;
    const u32 n_tables = sl.table_end - table0;
    const u32 per_table = (u32)std::max<u64>(1, std::min<u64>((entries + 255) / 256, std::max<u64>(1, 4096 / ((u64)n_tables * limbs))));
    for (u32 t = 0; t < n_tables; t += 32768) {  // (the grid's second dimension is limited to 65535)
        hipLaunchKernelGGL(gather_digits_kernel<V>, dim3(per_table, std::min<u32>(n_tables - t, 32768), limbs), dim3(256), 0, s, ctx->digits,
                           plan->tiles_s_dev, plan->wbase_s_dev, plan->owners_dev + table0 + t, limbs, plan->off_dev, plan->term_pt_dev, pt, wtab,
                           sl.tab_words, sl.tab_skip, sl.t_begin, sl.t_end, short_sums ? BLOCK_TERMS : CHUNK_TERMS);
    }
    const MacArgs<V> a{plan->digit_tiles_dev, plan->lists_dev, wtab, sl.tab_words, sl.tab_skip, ct_in, bias, out, limbs, ctx->N, sl.t_begin,
                       sl.t_end, mode};
    auto launch_form = [&](auto short_form) {
        constexpr bool SHORT = decltype(short_form)::value;
        if (mac_groups_stream(plan, limbs, ctx->N, sizeof(V))) launch_classes<V, SHORT, true>(ctx, a, c, blocks, s);
        else launch_classes<V, SHORT, false>(ctx, a, c, blocks, s);
    };
    if constexpr (sizeof(V) == sizeof(u64)) {
        if (short_sums) launch_form(std::true_type{});
    }
    if (!short_sums) launch_form(std::false_type{});
    HE_HIP(hipGetLastError());
    return HE_OK;
}

}  // namespace

// an upper bound of the workgroups that launch_mac_digits starts for the whole plan in either form, but for windows abreast (nine of
// them go as three runs of four): that form is checked where it is chosen
u64 mac_digits_blocks(const he_ctx* ctx, const he_plan* plan, u32 limbs) {
    u64 blocks = 0;
    for (u32 cls = 1; cls < SCALAR_CLASSES; cls++)
        blocks += mac_class_of<u64>(ctx, plan, limbs, cls, plan->class_begin_s[cls], plan->class_begin_s[cls + 1], ~0u).blocks;
    return blocks;
}

// groups of a class that a workgroup runs through, in a launch of the whole plan from the first term on, and whether they go abreast
u32 mac_digits_groups_per_workgroup(const he_ctx* ctx, const he_plan* plan, u32 limbs, u32 cls, bool packed, bool* abreast) {
    const u32 first = plan->class_begin_s[cls], end = plan->class_begin_s[cls + 1];
    const bool alone = plan->n_tiles_s - plan->class_begin_s[1] == end - first;
    MacClass m = packed ? mac_class_of<u32>(ctx, plan, limbs, cls, first, end, 0) : mac_class_of<u64>(ctx, plan, limbs, cls, first, end, 0);
    *abreast = !packed && alone && first < end &&
               go_abreast<u64>(ctx, plan, limbs, cls, first, end, 0, (u32)plan->table_end.size() - plan->table_s[first], m);
    return m.per_wg;
}

int launch_mac_digits(he_ctx* ctx, const he_plan* plan, const ScalarSlice& sl, u32 limbs, const u64* ct_in, const u64* pt, const u64* bias,
                      u64* out, u64* wtab, u32 mode, hipStream_t s) {
    return launch_mac_digits_t<u64>(ctx, plan, sl, limbs, ct_in, pt, bias, out, wtab, mode, s);
}

int launch_mac_digits32(he_ctx* ctx, const he_plan* plan, const ScalarSlice& sl, u32 limbs, const u32* ct_in, const u64* pt, const u64* bias,
                        u32* out, u64* wtab, u32 mode, hipStream_t s) {
    return launch_mac_digits_t<u32>(ctx, plan, sl, limbs, ct_in, pt, bias, out, wtab, mode, s);
}
