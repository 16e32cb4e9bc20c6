// The register-resident negacyclic transform's geometry and data movement, shared by the 64-bit and the packed
// 32-bit kernels: which index a register of a thread holds in each pass, the regrouping of the residues through
// the LDS between passes, and the loading of a pass's twiddles.  The butterflies themselves are the residue
// width's own (he_ntt.hip, he_packed32.hip).
//
// One workgroup transforms one polynomial limb (N residues).  Each of the T = N/16 threads keeps
// 16 residues in registers and runs up to four butterfly stages on them (a "pass") before the
// workgroup regroups the residues through LDS for the next pass.  Stage s (s = 0 .. log2N-1) pairs
// indices that differ in bit log2N-1-s, so pass p owns index bits [log2N-1-4p .. log2N-4-4p]; the
// last pass owns what is left at the bottom (1..4 stages) plus, to fill its 16 registers, the top
// bits again, so that consecutive threads hold consecutive short runs and global stores stay dense.
// A twiddle that is the same for the whole wavefront is read through the constant address space: a scalar
// load into scalar registers (the tables are never written by a kernel).  It takes no vector register, and it
// does not queue behind the vector stores of the previous row as a vector load would.
#pragma once
#include <type_traits>

#include "he_arith.h"

namespace {

template <int LOGN>
struct Geo {
    static constexpr int N = 1 << LOGN;
    static constexpr int T = N / 16;
    static constexpr int NPASS = (LOGN + 3) / 4;
    static constexpr int REM = LOGN - 4 * (NPASS - 1);  // stages of the last pass, 1..4
    static constexpr int LAST = NPASS - 1;
    // The orders of the accesses to rows in bit-reversed order: the last pass's, or MEMORY (see reg_index) where that leaves a
    // lane more than 16 bytes in a row; the loads of 32 bytes of 64-bit residues are not worth the regrouping (inverse
    // transforms of 4096 rows of 2^14: 336 us without, 340 with it; stores of forward ones 305 without, 298 with it).
    static constexpr int MEMORY = NPASS;
    static constexpr int STORE = REM > 1 ? MEMORY : LAST, LOAD = REM > 2 ? MEMORY : LAST;
    static constexpr int PACKED = REM > 2 ? MEMORY : LAST;  // 32-bit residues
};

// Index of register e of thread tid while pass P is being computed.  In the last pass the registers
// own the lowest REM index bits (the stages left) and, to fill 16 registers, the 4-REM bits just above
// the six bits that the lane number owns, so that a wavefront holds one aligned block of 1024.
// In the order MEMORY, in which rows in bit-reversed order are read and written, a lane holds two consecutive residues and
// its neighbours the next ones: an access of 16 bytes per lane is 1 KiB in one piece.  It is the last pass's own order when
// that has one stage; otherwise a regrouping within the wavefront lies between the two.  (In the last pass's order a lane
// holds 2^REM consecutive residues, and an instruction touches a part of every one of up to 64 cache lines: a rescale of 2048
// ciphertexts of N = 2^12 at L = 4 315 us, 268 in this order.)
template <int LOGN, int P>
__host__ __device__ constexpr u32 reg_index(u32 tid, u32 e) {
    using G = Geo<LOGN>;
    if constexpr (P < G::NPASS - 1) {
        constexpr int low = LOGN - 4 * (P + 1);
        u32 hi = tid >> low, lo = tid & ((1u << low) - 1);
        return (hi << (low + 4)) | (e << low) | lo;
    } else if constexpr (P == G::MEMORY) {
        return ((tid >> 6) << 10) | ((e >> 1) << 7) | ((tid & 63u) << 1) | (e & 1u);
    } else if constexpr (G::REM == 4) {
        return (tid << 4) | e;
    } else {
        u32 e_hi = e >> G::REM, e_lo = e & ((1u << G::REM) - 1);
        u32 wave = tid >> 6, lane = tid & 63u;
        return (wave << 10) | (e_hi << (G::REM + 6)) | (lane << G::REM) | e_lo;
    }
}

// The element of a row in memory that register e of thread tid holds in pass P.  The index is the thread's part plus the
// register's (disjoint bits): the row and the register's part are the same for the wave and make a scalar address, the
// thread's part is one 32-bit offset for all sixteen accesses.  (As one index per access they cost up to three vector
// instructions and two registers each.)
template <int LOGN, int P, typename V>
__device__ __forceinline__ V& row_at(V* row, u32 tid, u32 e) {
    typedef typename std::conditional<std::is_const<V>::value, const char, char>::type byte;
    return *reinterpret_cast<V*>(reinterpret_cast<byte*>(row + reg_index<LOGN, P>(0, e)) + reg_index<LOGN, P>(tid, 0) * (u32)sizeof(V));
}

// All sixteen registers of a thread from or to a row, in the order of pass P.  STREAM accesses (a choice that is the same for
// the whole launch) are marked as not to be kept in the caches: see the launchers for when.
template <int LOGN, int P>
__device__ __forceinline__ void load_row(u64 (&a)[16], const u64* row, u32 tid, bool stream) {
    if (stream) {
        asm volatile("; streamed loads" ::: "memory");  // (left to itself the compiler makes one loop of the two, of ordinary loads)
#pragma unroll
        for (u32 e = 0; e < 16; e++) a[e] = __builtin_nontemporal_load(&row_at<LOGN, P>(row, tid, e));
        asm volatile("; end" ::: "memory");
    } else {
#pragma unroll
        for (u32 e = 0; e < 16; e++) a[e] = row_at<LOGN, P>(row, tid, e);
    }
}
template <int LOGN, int P>
__device__ __forceinline__ void store_row(const u64 (&a)[16], u64* row, u32 tid, bool stream) {
    if (stream) {
        asm volatile("; streamed stores" ::: "memory");
#pragma unroll
        for (u32 e = 0; e < 16; e++) __builtin_nontemporal_store(a[e], &row_at<LOGN, P>(row, tid, e));
        asm volatile("; end" ::: "memory");
    } else {
#pragma unroll
        for (u32 e = 0; e < 16; e++) row_at<LOGN, P>(row, tid, e) = a[e];
    }
}

// True when, in pass P, every wavefront (64 consecutive threads) holds exactly the aligned block of
// 1024 indices with its own number: a regrouping between two such passes moves data only within
// wavefronts.  Checked over all threads and registers at compile time.
template <int LOGN, int P>
constexpr bool wave_holds_own_block() {
    for (u32 tid = 0; tid < (u32)Geo<LOGN>::T; tid++)
        for (u32 e = 0; e < 16; e++)
            if ((reg_index<LOGN, P>(tid, e) >> 10) != (tid >> 6)) return false;
    return true;
}

// LDS placement: one slot of padding after every sixteen, so that the strided access patterns of the regrouping steps
// spread over the banks (64-bit residues: no conflict in any pass of any ring degree; 32-bit ones two-way conflicts in some).
// An aligned block of 1024 indices keeps a range of slots of its own.  Of two indices without common bits the slot of the
// sum is the sum of the slots: an access is one base per thread and a constant that goes into the instruction.  (As an
// exclusive or of index bits the placement cost an instruction per access, 96 of about 1900 in a transform of 2^14.)
__host__ __device__ constexpr u32 lds_slot(u32 idx) { return idx + (idx >> 4); }

// bytes of a row of N residues of type V in the LDS
template <int LOGN, typename V>
constexpr u32 lds_row_bytes() { return lds_slot(Geo<LOGN>::N) * (u32)sizeof(V); }

// Workgroup barrier that orders LDS traffic only: waits for this wave's LDS operations, then for the
// other waves.  (A full __syncthreads() would also wait for outstanding global loads, and the
// twiddles of the next pass are deliberately in flight across the regrouping.)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The same for data that stays within one wavefront: the LDS serves a wave's operations in the order
// they were issued, so the wave only has to keep that order (and nothing may be moved across by the
// compiler); other waves are not waited for and run ahead or behind freely.
__device__ __forceinline__ void lds_wave_order() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Where a thread's registers of pass P are in the LDS.  (An instruction's constant offset reaches 64 KiB; the first pass of
// N = 2^14 has accesses beyond that, which take an addition.)
template <typename V, int LOGN, int P>
struct LdsBase {
    typedef __attribute__((address_space(3))) V lds_v;
    static constexpr u32 offset(u32 e) { return lds_slot(reg_index<LOGN, P>(0, e)) * (u32)sizeof(V); }
    u32 base;
    __device__ __forceinline__ LdsBase(V* row, u32 tid) {
        base = (u32)(uintptr_t)(lds_v*)row + lds_slot(reg_index<LOGN, P>(tid, 0)) * (u32)sizeof(V);
        asm("" : "+v"(base));  // (else the constants are added to the row's address, one instruction and register each)
    }
    __device__ __forceinline__ lds_v* operator()(u32 e) const { return (lds_v*)(uintptr_t)(base + offset(e)); }
};

// (V: the residue type, u64 or u32; the row in the LDS is N of them)
template <int LOGN, int PFROM, int PTO, typename V>
__device__ __forceinline__ void regroup(V (&a)[16], V* lds, u32 tid) {
    constexpr bool WAVE_LOCAL = wave_holds_own_block<LOGN, PFROM>() && wave_holds_own_block<LOGN, PTO>();
    // reg_index(tid, e) = reg_index(tid, 0) + reg_index(0, e) (disjoint bits), and so are their slots: see lds_slot
    // The two bases are derived from copies of the thread index that the optimizer cannot relate to
    // each other or to other passes: a regrouping writes where the previous one read, and addresses
    // kept alive from one to the next would cost more registers than the few operations they save.
    u32 tid_w = tid, tid_r = tid;
    asm("; regroup %1 write" : "+v"(tid_w) : "n"(PFROM * 16 + PTO));
    asm("; regroup %1 read" : "+v"(tid_r) : "n"(PFROM * 16 + PTO));
    // earlier readers of the slots written here are done: all waves, or (wave-local) this wave only,
    // since its block of slots is then touched by no other wave until the next workgroup-wide regrouping
    if constexpr (WAVE_LOCAL) lds_wave_order(); else lds_barrier();
    {
        const LdsBase<V, LOGN, PFROM> at(lds, tid_w);
#pragma unroll
        for (u32 e = 0; e < 16; e++) *at(e) = a[e];
    }
    if constexpr (WAVE_LOCAL) lds_wave_order(); else lds_barrier();
    {
        const LdsBase<V, LOGN, PTO> at(lds, tid_r);
#pragma unroll
        for (u32 e = 0; e < 16; e++) a[e] = *at(e);
    }
}

// ... if the two orders differ (between the last pass's and that of the accesses to memory)
template <int LOGN, int FROM, int TO, typename V>
__device__ __forceinline__ void reorder(V (&a)[16], V* lds, u32 tid) {
    if constexpr (FROM != TO) regroup<LOGN, FROM, TO>(a, lds, tid);
}

// Tw: the twiddle type, Twiddle (two 64-bit words), Twiddle32 (two 32-bit words) or TwiddleF (one double): a table
// entry as it is stored.  For the two-word types Tw::raw is a vector type of the same layout, through which a
// wave-uniform entry is read with a scalar load.
template <typename Tw, bool UNIFORM>
__device__ __forceinline__ Tw load_twiddle(const Tw* tw, u32 k) {
    if constexpr (__is_same(Tw, TwiddleF)) {  // one double per entry
        if constexpr (UNIFORM) {
            k = __builtin_amdgcn_readfirstlane(k);
            return Tw{*(const __attribute__((address_space(4))) double*)(tw + k)};
        } else {
            return tw[k];
        }
    } else {
        typedef typename Tw::raw raw;
        static_assert(sizeof(raw) == sizeof(Tw), "a table entry is a pair of words");
        raw v;
        if constexpr (UNIFORM) {
            k = __builtin_amdgcn_readfirstlane(k);
            v = *(const __attribute__((address_space(4))) raw*)(tw + k);
        } else {
            v = *reinterpret_cast<const raw*>(tw + k);
        }
        return Tw{v.x, v.y};
    }
}

// Shape of pass P: its stages, and where the twiddle of (stage k, register e) sits among the
// pass's twiddles.  A thread's twiddles of stage k are 2^k consecutive table entries (per group of
// registers in the last pass), 15 entries per pass at most.
template <int LOGN, int P>
struct PassShape {
    using G = Geo<LOGN>;
    static constexpr bool LAST = (P == G::NPASS - 1);
    static constexpr int NST = LAST ? G::REM : 4;
    static constexpr int GROUPS = 16 >> NST;                 // independent register groups (last pass only > 1)
    static constexpr int PER_GROUP = (1 << NST) - 1;
    static constexpr int COUNT = GROUPS * PER_GROUP;
    // twiddles are the same for the whole wave when the thread-dependent part of the group index
    // is constant over 64 consecutive threads
    static constexpr bool UNIFORM = (P == 0) || (!LAST && (LOGN - 4 * (P + 1)) >= 6);
    __device__ static constexpr int slot(int k, u32 e) {
        return (int)(e >> NST) * PER_GROUP + ((1 << k) - 1) + (int)((e & ((1u << NST) - 1)) >> (NST - k));
    }
};

template <int LOGN, int P, typename Tw = Twiddle>
struct PassTwiddles {
    Tw t[PassShape<LOGN, P>::COUNT];
};

// The twiddles of stages K0 .. K1 - 1 of pass P for this thread, requested in one go (all of a pass's: the caller does
// this before the regrouping that precedes the pass, so the loads overlap the LDS traffic).
template <int LOGN, int P, int K0 = 0, int K1 = PassShape<LOGN, P>::NST, typename Tw>
__device__ __forceinline__ void load_pass_twiddles(PassTwiddles<LOGN, P, Tw>& pt, const Tw* tw, u32 tid) {
    using S = PassShape<LOGN, P>;
    asm("; twiddles of pass %1" : "+v"(tid) : "n"(P));  // addresses are derived here, not ahead of earlier passes
#pragma unroll
    for (int k = K0; k < K1; k++) {
        const int s = 4 * P + k;
        const int bit = S::NST - 1 - k;
#pragma unroll
        for (u32 e = 0; e < 16; e++) {
            if (e & (1u << bit)) continue;
            if ((e & ((1u << S::NST) - 1)) & ((1u << bit) - 1)) continue;  // one load per distinct twiddle
            const u32 j = reg_index<LOGN, P>(tid, e);
            pt.t[S::slot(k, e)] = load_twiddle<Tw, S::UNIFORM>(tw, (1u << s) + (j >> (LOGN - s)));
        }
    }
}

// A copy of the thread index that the optimizer treats as a new value: addresses derived from it
// are computed where they are used instead of being carried (in registers the transform needs)
// from the top of the kernel.
__device__ __forceinline__ u32 fresh(u32 tid) {
    asm("; fresh thread index" : "+v"(tid));
    return tid;
}

}  // namespace
