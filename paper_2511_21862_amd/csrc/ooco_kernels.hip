// HIP kernels of libooco for gfx950 (CDNA4, wave64): split-KV decode attention with its in-kernel
// merge, prefill-chunk attention and KV block copy.
//
// Common scheme (decode and prefill): scores are computed TRANSPOSED, S^T[token][query column]
// = K · Q^T, and the output as O^T[dim][query column] = V^T · P^T.  A "query column" is a query
// head of the GQA group (decode) or a query row (prefill).  With the MFMA operand/result lane
// layouts this keeps one query column in one lane column for the whole kernel:
//   * the fp32 result of the first MFMA is, register for register, the B operand of the second
//     one (after bf16 rounding) -- no cross-lane movement of P;
//   * the softmax statistics (max, sum) and the accumulator rescale are per lane column;
//   * K tiles [hd/8][16][8] and V tiles [hd][16] of the paged cache are already in A-operand
//     order, so they go from global memory straight into MFMA source registers (decode) or are
//     copied unchanged into LDS by direct global->LDS loads and read from there (prefill).
// Softmax runs in base 2: scores are multiplied by scale*log2(e) and exponentiated with
// v_exp_f32.  Masked scores are set to -inf by select; V values of slots past the end of a
// sequence are zeroed by select (those slots may hold NaN/Inf).
#include "ooco_internal.h"

#include <algorithm>
#include <cfloat>
#include <type_traits>

namespace ooco {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define OOCO_DEV __device__ __forceinline__

constexpr int kNoVmem = 0x78F;   // sched_barrier mask: everything but vector-memory operations may cross

OOCO_DEV uint32_t pack2_bf16(float a, float b)
{
    bf16x2 v = {(__bf16)a, (__bf16)b};   // round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}

OOCO_DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max of three without the NaN-quieting moves that fmaxf would add (one v_max3_f32)
OOCO_DEV float max3(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// max of two / with a floor of -1e30, as single instructions (no NaN-quieting moves)
OOCO_DEV float max2(float a, float b)
{
    float d;
    asm("v_max_f32_e32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}
OOCO_DEV float floor_m1e30(float a)
{
    float d;
    asm("v_max_f32_e32 %0, 0xf149f2ca, %1" : "=v"(d) : "v"(a));   // 0xf149f2ca = -1e30f
    return d;
}
// max of the 32 scores a lane holds for one step (two 16-register MFMA results), as one dependent chain of
// v_max3_f32 in two asm statements (an asm statement takes at most 30 operands)
OOCO_DEV float max32(const f32x16 &a, const f32x16 &b)
{
    float d, e;
    asm("v_max3_f32 %0, %1, %2, %3\n\t"
        "v_max3_f32 %0, %0, %4, %5\n\t"
        "v_max3_f32 %0, %0, %6, %7\n\t"
        "v_max3_f32 %0, %0, %8, %9\n\t"
        "v_max3_f32 %0, %0, %10, %11\n\t"
        "v_max3_f32 %0, %0, %12, %13\n\t"
        "v_max3_f32 %0, %0, %14, %15\n\t"
        "v_max3_f32 %0, %0, %16, %17"
        : "=&v"(d)
        : "v"(a[0]), "v"(b[0]), "v"(a[1]), "v"(b[1]), "v"(a[2]), "v"(b[2]), "v"(a[3]), "v"(b[3]), "v"(a[4]), "v"(b[4]),
          "v"(a[5]), "v"(b[5]), "v"(a[6]), "v"(b[6]), "v"(a[7]), "v"(b[7]), "v"(a[8]));
    asm("v_max3_f32 %0, %1, %2, %3\n\t"
        "v_max3_f32 %0, %0, %4, %5\n\t"
        "v_max3_f32 %0, %0, %6, %7\n\t"
        "v_max3_f32 %0, %0, %8, %9\n\t"
        "v_max3_f32 %0, %0, %10, %11\n\t"
        "v_max3_f32 %0, %0, %12, %13\n\t"
        "v_max3_f32 %0, %0, %14, %15\n\t"
        "v_max_f32_e32 %0, %0, %16"
        : "=&v"(e)
        : "v"(d), "v"(b[8]), "v"(a[9]), "v"(b[9]), "v"(a[10]), "v"(b[10]), "v"(a[11]), "v"(b[11]), "v"(a[12]), "v"(b[12]),
          "v"(a[13]), "v"(b[13]), "v"(a[14]), "v"(b[14]), "v"(a[15]), "v"(b[15]));
    return e;
}

// the same of 16 scores
OOCO_DEV float max16(const f32x16 &a)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3\n\t"
        "v_max3_f32 %0, %0, %4, %5\n\t"
        "v_max3_f32 %0, %0, %6, %7\n\t"
        "v_max3_f32 %0, %0, %8, %9\n\t"
        "v_max3_f32 %0, %0, %10, %11\n\t"
        "v_max3_f32 %0, %0, %12, %13\n\t"
        "v_max3_f32 %0, %0, %14, %15\n\t"
        "v_max_f32_e32 %0, %0, %16"
        : "=&v"(d)
        : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]), "v"(a[9]),
          "v"(a[10]), "v"(a[11]), "v"(a[12]), "v"(a[13]), "v"(a[14]), "v"(a[15]));
    return d;
}

// acc + lo + hi of a packed bf16 pair (one v_dot2c_f32_bf16 against the pair (1, 1))
OOCO_DEV float sum2_bf16(uint32_t pair, float acc)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, 0x3F803F80u), acc,
                                           false);
}

// Device-scope (all XCDs) relaxed store / load of one float: the store writes through to memory,
// the load bypasses the non-coherent cache levels.
typedef float f32x2 __attribute__((ext_vector_type(2)));
OOCO_DEV void store_dev2(float *ptr, float a, float b)   // ptr is 8-byte aligned
{
    const f32x2 v = {a, b};
    __hip_atomic_store(reinterpret_cast<uint64_t *>(ptr), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
// The same cache policy for a 16-byte store (a plain vector store with the device-scope bit: the ordering
// against the arrival counter comes from s_waitcnt, 16-byte atomicity is not needed).  Far fewer memory
// operations than 8-byte atomic stores, which matters for the 64 KiB partial results of a prefill part.
// (The s_nop covers the wait states a wide store needs before its data registers may be overwritten, which
// the compiler cannot see through the asm.)
OOCO_DEV void store_dev4(float *ptr, f32x4 v)   // ptr is 16-byte aligned
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(ptr), "v"(v) : "memory");
}
// Sixteen device-scope 16-byte loads of a lane, N (1 KiB apart) from each of 16 / N pointers: pieces of the parts of a split
// prefill tile.  All loads and the wait for them sit in ONE asm statement, so that the compiler never sees a register it
// believes loaded while the data is still on its way.
#define OOCO_LD4(o, a) \
    "global_load_dwordx4 %" #o ", %" #a ", off sc1\n\t"
#define OOCO_LD4O(o, a, off) \
    "global_load_dwordx4 %" #o ", %" #a ", off offset:" #off " sc1\n\t"
template <int N>
OOCO_DEV void load_dev_part(f32x4 (&t)[16], const float *p0, const float *p1, const float *p2, const float *p3)
{
    static_assert(N == 4, "sixteen loads");
    asm volatile(OOCO_LD4(0, 16) OOCO_LD4O(1, 16, 1024) OOCO_LD4O(2, 16, 2048) OOCO_LD4O(3, 16, 3072)
                 OOCO_LD4(4, 17) OOCO_LD4O(5, 17, 1024) OOCO_LD4O(6, 17, 2048) OOCO_LD4O(7, 17, 3072)
                 OOCO_LD4(8, 18) OOCO_LD4O(9, 18, 1024) OOCO_LD4O(10, 18, 2048) OOCO_LD4O(11, 18, 3072)
                 OOCO_LD4(12, 19) OOCO_LD4O(13, 19, 1024) OOCO_LD4O(14, 19, 2048) OOCO_LD4O(15, 19, 3072)
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7]),
                   "=&v"(t[8]), "=&v"(t[9]), "=&v"(t[10]), "=&v"(t[11]), "=&v"(t[12]), "=&v"(t[13]), "=&v"(t[14]), "=&v"(t[15])
                 : "v"(p0), "v"(p1), "v"(p2), "v"(p3)
                 : "memory");
}
template <int N>
OOCO_DEV void load_dev_part(f32x4 (&t)[16], const float *p0, const float *p1, const float *p2, const float *p3, const float *p4,
                            const float *p5, const float *p6, const float *p7)
{
    static_assert(N == 2, "sixteen loads");
    asm volatile(OOCO_LD4(0, 16) OOCO_LD4O(1, 16, 1024) OOCO_LD4(2, 17) OOCO_LD4O(3, 17, 1024)
                 OOCO_LD4(4, 18) OOCO_LD4O(5, 18, 1024) OOCO_LD4(6, 19) OOCO_LD4O(7, 19, 1024)
                 OOCO_LD4(8, 20) OOCO_LD4O(9, 20, 1024) OOCO_LD4(10, 21) OOCO_LD4O(11, 21, 1024)
                 OOCO_LD4(12, 22) OOCO_LD4O(13, 22, 1024) OOCO_LD4(14, 23) OOCO_LD4O(15, 23, 1024)
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(t[4]), "=&v"(t[5]), "=&v"(t[6]), "=&v"(t[7]),
                   "=&v"(t[8]), "=&v"(t[9]), "=&v"(t[10]), "=&v"(t[11]), "=&v"(t[12]), "=&v"(t[13]), "=&v"(t[14]), "=&v"(t[15])
                 : "v"(p0), "v"(p1), "v"(p2), "v"(p3), "v"(p4), "v"(p5), "v"(p6), "v"(p7)
                 : "memory");
}
#undef OOCO_LD4
#undef OOCO_LD4O
OOCO_DEV f32x2 load_dev2(const float *ptr)
{
    const uint64_t u = __hip_atomic_load(reinterpret_cast<uint64_t *>(const_cast<float *>(ptr)), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    return __builtin_bit_cast(f32x2, u);
}


// ------------------------------------------------------------------------------------------
// Cross-lane reductions over the four 16-lane rows of a wave with the CDNA4 lane-swap
// instructions (VALU only, no LDS traffic): v_permlane16_swap exchanges the odd rows of its first
// operand with the even rows of the second, v_permlane32_swap the upper half of the first with
// the lower half of the second; fed with two copies of one value they return both partners of
// an xor-16 / xor-32 butterfly.  (Vector elements are copied to scalars before
// __builtin_bit_cast: a bit_cast applied directly to an element reference reads element 0.)
OOCO_DEV void swap16(float v, float &lo, float &hi)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned a0 = a[0], a1 = a[1];
    lo = __builtin_bit_cast(float, a0);
    hi = __builtin_bit_cast(float, a1);
}
OOCO_DEV void swap32(float v, float &lo, float &hi)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned a0 = a[0], a1 = a[1];
    lo = __builtin_bit_cast(float, a0);
    hi = __builtin_bit_cast(float, a1);
}
OOCO_DEV float rows_max(float v)
{
    float x, y;
    swap16(v, x, y);
    swap32(fmaxf(x, y), x, y);
    return fmaxf(x, y);
}
OOCO_DEV float rows_sum(float v)
{
    float x, y;
    swap16(v, x, y);
    swap32(x + y, x, y);
    return x + y;
}

// ------------------------------------------------------------------------------------------
// Work lookup shared by both kernels: cum[] is non-decreasing with cum[0] = 0; returns the number
// of entries j in [1, n] with cum[j] <= x, i.e. the index i with cum[i] <= x < cum[i+1].
// All 64 lanes of the wave must call it with the same x.
template <class CumAt>
OOCO_DEV int count_le(CumAt cum_at, int n, int x, int lane)
{
    int cnt = 0;
    for (int base = 1; base <= n; base += 64) {
        const int idx = base + lane;
        const int v = idx <= n ? cum_at(idx) : 0x7FFFFFFF;
        const int c = __popcll(__ballot(v <= x));
        cnt += c;
        if (c < 64) break;
    }
    return cnt;
}

// ------------------------------------------------------------------------------------------
// Equal runs of the decode line (RunLayout without XCD weights and tail, which only decode_kernel_general works on): the same
// numbers as run_bounds and run_of by the reciprocal in double precision and an exact remainder.  The compiler's 64-bit
// divisions -- a branch to a short and a long form each, and with the weighted form inlined eight of them per call -- made the
// first 1100 instructions of a decode wave, and instruction fetch is what a small launch starts with.
struct EqualRuns {
    int32_t blocks, runs;
    static OOCO_DEV double reciprocal(int n)   // 1 / n to the last place or two
    {
        const double d = (double)n, r0 = __builtin_amdgcn_rcp(d);
        const double r1 = __builtin_fma(__builtin_fma(-d, r0, 1.0), r0, r0);
        return __builtin_fma(__builtin_fma(-d, r1, 1.0), r1, r1);
    }
    static OOCO_DEV int quotient(int a, int b, int c, int n, double inv)   // wave-uniform
    {
        return __builtin_amdgcn_readfirstlane(quotient_by_reciprocal(a, b, c, n, inv));
    }
    OOCO_DEV void bounds(int run, int &lo, int &hi) const
    {
        const double inv = reciprocal(runs);
        lo = quotient(blocks, run, 0, runs, inv);
        hi = quotient(blocks, run + 1, 0, runs, inv);
    }
    // runs that hold units x and y
    OOCO_DEV void holding(int x, int y, int &rx, int &ry) const
    {
        const double inv = reciprocal(blocks);
        rx = quotient(x + 1, runs, 1, blocks, inv);
        ry = quotient(y + 1, runs, 1, blocks, inv);
    }
};
struct GeneralRuns {
    RunLayout L;
    OOCO_DEV void bounds(int run, int &lo, int &hi) const { run_bounds(L, run, lo, hi); }
    OOCO_DEV void holding(int x, int y, int &rx, int &ry) const
    {
        rx = run_of(L, x);
        ry = run_of(L, y);
    }
};

// The sequence i with cum[i] <= x < cum[i + 1], and those two values.  head: lane l holds cum[l + 1] (anything for l >= n),
// loaded with the kernel's first loads; what it does not reach is read here.
template <class CumAt>
OOCO_DEV int locate(CumAt cum_at, int head, int n, int x, int lane, int &cs, int &ce)
{
    int before = 0;   // cum[base - 1]
    for (int base = 1;; base += 64) {
        const int idx = base + lane;
        const int v = idx > n ? 0x7FFFFFFF : base == 1 ? head : cum_at(idx);
        const int c = __popcll(__ballot(v <= x));
        if (c < 64) {
            cs = c ? __builtin_amdgcn_readlane(v, c - 1) : before;
            ce = __builtin_amdgcn_readlane(v, c);
            return base - 1 + c;
        }
        before = __builtin_amdgcn_readlane(v, 63);
    }
}

// ------------------------------------------------------------------------------------------
// Decode: one wave per (run k of the decode block line, kv head).  A wave walks the pieces of its
// run one after the other; a piece is a range of KV blocks of one sequence.  Per 16-token block:
//   S^T[16 tok][16 heads] = K[16 tok][hd] · Q^T[hd][16 heads]      (hd/32 x v_mfma_f32_16x16x32_bf16)
//   O^T[hd][16 heads]    += V^T[hd][16 tok] · P^T[16 tok][16 heads] (hd/16 x v_mfma_f32_16x16x16_bf16)
// Head columns >= g (the GQA group size) carry zeros.  Lane l = 16*kq + col:
//   K operand, chunk c:  16 B at tile offset (64c + l)*16          (token col, dims 32c+8kq..+8)
//   S^T result reg r:    token 4kq + r, head col
//   V operand, group nb: 8 B at tile offset ((16nb + col)*16 + 4kq)*2   (dim 16nb+col, tokens 4kq..+4)
//   O^T result reg r:    dim 16nb + 4kq + r, head col
// One K and one V register set: the K loads of block j+1 are issued right after the QK MFMAs of
// block j have consumed the K registers, the V loads of block j+1 right after the PV MFMAs, so a
// wave always has one block's tiles (8 KiB with head_dim 128) on their way; a few such waves per
// compute unit keep HBM busy, and no second register set is needed.
//
// A piece that covers its whole sequence normalises and stores bf16 output.  Any other piece
// stores (acc, m, l) in fp32 into partial slot k + seq, then bumps the arrival counter of
// (seq, kv head); the piece that arrives last merges all slots of the sequence in slot order
// (so the result does not depend on which piece is last) and resets the counter.

// The blocks [blk_begin, blk_begin + nblk) of sequence seq (not none) against its query row, streamed by wave `wave` of NW
// waves that take steps of NBI blocks in turn: un-normalised output O, running maximum m (the same in the four rows of a
// lane column) and this lane's share lsum of the sum, as laid out above.  A wave without a step has (0, -inf, 0), one whose
// scores are all -inf (0, -FLT_MAX, 0); neither weighs anything beside one with a score.
// q_row: the sequence's query row, read here (after the block ids have been asked for: one memory round trip for both).
template <int HD, int NBI, int NW>
OOCO_DEV void decode_stream(const AttnParams &p, int kvh, int seq, int blk_begin, int nblk, int &q_row, int wave,
                            int lane, uint64_t *trace, bool &first_piece, f32x4 (&O)[HD / 16], float &m, float &lsum)
{
    constexpr int KC = HD / 32;
    constexpr int NB = HD / 16;
    const int col = lane & 15;
    const int kq = lane >> 4;
    const int g = p.g;
    const int64_t tile_elems = (int64_t)HD * kBlockSize;   // one (block, kv head) tile
    const int head = kvh * g + col;
    const int nstep = ((nblk + NBI - 1) / NBI - wave + NW - 1) / NW;   // of this wave
    // block (of the piece) that is this wave's i-th
    auto blk_of = [&](int i) -> int { return NW == 1 ? i : (i / NBI * NW + wave) * NBI + i % NBI; };

    // rolling window of the physical ids of this wave's next 64 blocks, one per lane
    const int32_t *table = p.block_tables + (int64_t)seq * p.max_blocks_per_seq + blk_begin;
    int wbase = 0;
    int idv = table[min(blk_of(lane), nblk - 1)];
    int idn = table[min(blk_of(64 + lane), nblk - 1)];
    const int q_raw = p.query_start_loc[seq], seq_len = p.seq_lens[seq];
    // (sent off together, before anything waits for one of them)
    __builtin_amdgcn_sched_barrier(kNoVmem);
    q_row = min(max(q_raw, 0), p.total_q - 1);
    if (NW > 1 && nstep <= 0) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) O[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
        m = -INFINITY;
        lsum = 0.f;
        return;
    }
    // Q as B operand: head col, dims 32c + 8kq .. +8
    u32x4 qb[KC];
    {
        const u32x4 *qp = reinterpret_cast<const u32x4 *>(p.q + ((int64_t)q_row * p.Hq + (col < g ? head : 0)) * HD);
#pragma unroll
        for (int c = 0; c < KC; ++c) {
            u32x4 t = qp[c * 4 + kq];
            qb[c] = (col < g) ? t : u32x4{0u, 0u, 0u, 0u};
        }
    }
    u32x4 kreg[NBI][KC];
    u32x2 vreg[NBI][NB];
    int64_t offs[NBI];
    auto tile_off = [&](int j) -> int64_t {   // j (of this wave's blocks) is wave-uniform and non-decreasing
        if (j - wbase >= 64) {
            wbase += 64;
            idv = idn;
            asm volatile("" : "+v"(idv));   // (waited for here, in the rare path, and not where the ids are used)
            idn = table[min(blk_of(wbase + 64 + lane), nblk - 1)];
        }
        const int pb = __builtin_amdgcn_readlane(idv, j - wbase);
        return ((int64_t)pb * p.Hkv + kvh) * tile_elems;
    };
    // K and V tiles are read once per kv head and never again in this launch: they are loaded with the
    // non-temporal policy (`nt`), so that the stream does not push other data out of the caches on its way
    // through them.  Measured on MI355X: 64 sequences 115.7 -> 103.3 us, 512 sequences 1.149 -> 1.030 ms
    // (6.1 -> 6.8 TB/s).
    // Loads are issued unconditionally (steps past the end re-read the last block, an L2 hit)
    // so that every step has the same number of loads in flight and the waits before the
    // MFMAs can leave the younger loads outstanding.
    auto issue_k = [&](int step) {
#pragma unroll
        for (int u = 0; u < NBI; ++u) {
            offs[u] = tile_off(min(step * NBI + u, NW == 1 ? nblk - 1 : nstep * NBI - 1));
            const u32x4 *kp = reinterpret_cast<const u32x4 *>(p.k_cache + offs[u]);
#pragma unroll
            for (int c = 0; c < KC; ++c) kreg[u][c] = __builtin_nontemporal_load(&kp[c * 64 + lane]);
        }
    };
    auto issue_v = [&]() {
#pragma unroll
        for (int u = 0; u < NBI; ++u) {
            const u32x2 *vp = reinterpret_cast<const u32x2 *>(p.v_cache + offs[u]);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) vreg[u][nb] = __builtin_nontemporal_load(&vp[(nb * 16 + col) * 4 + kq]);
        }
    };

#pragma unroll
    for (int nb = 0; nb < NB; ++nb) O[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    m = -FLT_MAX;   // (finite: a first step whose scores all overflow to -inf weighs nothing, where -inf - -inf would make it NaN)
    lsum = 0.f;

    issue_k(0);
    // The K loads stay ahead of the V loads also here: the waits of the loop are the longest that either way into it
    // needs, and K loads that the scheduler moves behind V loads make every step wait for the V tiles before its scores.
    __builtin_amdgcn_sched_barrier(kNoVmem);
    issue_v();
    if (trace && first_piece) {   // time at which the first K/V tiles of the wave have arrived
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) trace[1] = wall_clock64();
        first_piece = false;
    }
    for (int t = 0; t < nstep; ++t) {
        f32x4 S[NBI];
#pragma unroll
        for (int u = 0; u < NBI; ++u) {
            S[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < KC; ++c)
                S[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kreg[u][c]),
                                                               __builtin_bit_cast(bf16x8, qb[c]), S[u], 0, 0, 0);
        }
        issue_k(min(t + 1, nstep - 1));
        float mloc = -INFINITY;
#pragma unroll
        for (int u = 0; u < NBI; ++u) {
            const int j = blk_of(t * NBI + u);
            int nvalid = seq_len - (blk_begin + j) * kBlockSize;
            if (NBI > 1 && j >= nblk) nvalid = 0;
            if (nvalid < kBlockSize) {   // wave-uniform: tail block of the sequence, or past the piece
#pragma unroll
                for (int r = 0; r < 4; ++r) S[u][r] = (4 * kq + r < nvalid) ? S[u][r] * p.scale_log2e : -INFINITY;
                const uint32_t m0 = (4 * kq + 0 < nvalid ? 0x0000FFFFu : 0u) | (4 * kq + 1 < nvalid ? 0xFFFF0000u : 0u);
                const uint32_t m1 = (4 * kq + 2 < nvalid ? 0x0000FFFFu : 0u) | (4 * kq + 3 < nvalid ? 0xFFFF0000u : 0u);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    vreg[u][nb][0] &= m0;
                    vreg[u][nb][1] &= m1;
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) S[u][r] *= p.scale_log2e;
            }
            mloc = fmaxf(mloc, fmaxf(fmaxf(S[u][0], S[u][1]), fmaxf(S[u][2], S[u][3])));
        }
        mloc = rows_max(mloc);
        const float m_new = fmaxf(m, mloc);
        const float alpha = fast_exp2(m - m_new);
        const bool grow = m_new > m;
        m = m_new;
        float psum = 0.f;
        s16x4 P[NBI];
#pragma unroll
        for (int u = 0; u < NBI; ++u) {
            float e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) e[r] = fast_exp2(S[u][r] - m_new);
            psum += (e[0] + e[1]) + (e[2] + e[3]);
            const u32x2 pk = {pack2_bf16(e[0], e[1]), pack2_bf16(e[2], e[3])};
            P[u] = __builtin_bit_cast(s16x4, pk);
        }
        lsum = lsum * alpha + psum;
        if (__any(grow)) {
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int r = 0; r < 4; ++r) O[nb][r] *= alpha;
        }
#pragma unroll
        for (int u = 0; u < NBI; ++u)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                O[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, vreg[u][nb]), P[u],
                                                                  O[nb], 0, 0, 0);
        issue_v();
    }
}

// One run of the decode line for one kv head, all its pieces, executed by one wave (see above).
// `at_stream_end()` is called once the last piece of the run has been streamed, before its epilogue.
template <int HD, int NBI, int MBATCH, class CumAt, class Runs, class AtStreamEnd>
OOCO_DEV void decode_run(const AttnParams &p, CumAt cum_at, int cum_head, const Runs &L, int run, int kvh, int lane, uint64_t *trace,
                         bool &first_piece, AtStreamEnd at_stream_end)
{
    constexpr int NB = HD / 16;
    const int col = lane & 15;
    const int kq = lane >> 4;
    const int g = p.g;
    const int head = kvh * g + col;
    int lo, hi;
    L.bounds(run, lo, hi);
    int cs, ce, pos = lo;
    int seq = locate(cum_at, cum_head, p.num_seqs, lo, lane, cs, ce);
    while (pos < hi) {
        while (ce <= pos) {   // the next sequence with decode blocks
            ++seq;
            cs = ce;
            ce = cum_at(seq + 1);
        }
        seq = __builtin_amdgcn_readfirstlane(seq);
        const int stop = min(hi, ce);
        // the sequence's blocks start piece_pad units into its stretch of the line
        const int first = cs + p.piece_pad;
        const int begin = max(pos, first);
        if (begin >= stop) {   // the run ends before the first block of this sequence
            if (trace && lane == 0) trace[2] = wall_clock64();
            pos = stop;
            continue;
        }
        const int blk_begin = begin - first;
        const int nblk = stop - begin;
        const bool whole = (begin == first) && (stop == ce);

        f32x4 O[NB];
        float m, lsum;
        int q_row;
        decode_stream<HD, NBI, 1>(p, kvh, seq, blk_begin, nblk, q_row, 0, lane, trace, first_piece, O, m, lsum);

        if (trace && stop == hi && lane == 0) trace[2] = wall_clock64();   // end of streaming
        if (stop == hi) at_stream_end();
        float ltot = rows_sum(lsum);
        bool store_out = whole;
        if (!whole) {
            // ---- partial result into slot run + seq, then arrival count.  Partials are written
            // and read with device-scope accesses (write-through / L2-bypassing), so that pieces
            // running on other XCDs see them without any whole-cache write-back or invalidate.
            if (col < g) {
                const int64_t row = (int64_t)(run + seq) * p.Hq + head;
                float *ap = p.part_acc + row * HD + 4 * kq;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) store_dev4(ap + nb * 16, O[nb]);
                if (kq == 0) store_dev2(p.part_ml + row * 2, m, ltot);
            }
            int first_run, last_run;
            L.holding(first, ce - 1, first_run, last_run);
            const int nparts = last_run - first_run + 1;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the partial has reached memory before the count
            int prev = 0;
            if (lane == 0)
                prev = __hip_atomic_fetch_add(p.counters + (int64_t)seq * p.Hkv + kvh, 1, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
            prev = __builtin_amdgcn_readfirstlane(prev);
            if (prev == nparts - 1) {   // last piece of this (sequence, kv head): merge, in slot order
                // The 16 lane columns hold only g heads, so 16/g (at most 4) groups of columns merge
                // different parts side by side: column group pg takes the parts pg, pg + ngrp, ...
                // (three at a time so that their memory round trips overlap); the groups' results
                // are then folded into group 0 in a fixed order.  Which parts meet in which order
                // depends only on the plan, never on which piece arrived last.
                // (only for sequences cut into many parts: below that one group is as fast and loads less)
                const int ngrp = nparts <= 2 * 3 ? 1 : (g <= 4 ? 4 : (g <= 8 ? 2 : 1));
                const int pg = col / g, hc = col - pg * g;
                const bool member = pg < ngrp;
                const int hm = kvh * g + (member ? hc : 0);
                float M = -INFINITY;
                ltot = 0.f;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) O[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
                auto fold = [&](float m2, float l2, const f32x4 (&o2)[NB]) {   // (M, ltot, O) <- merged with (m2, l2, o2)
                    const float M_new = fmaxf(M, m2);
                    const float w_old = fast_exp2(M - M_new), w_new = fast_exp2(m2 - M_new);
                    M = M_new;
                    ltot = ltot * w_old + l2 * w_new;
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) O[nb][r] = O[nb][r] * w_old + o2[nb][r] * w_new;
                };
                // (MBATCH parts per round trip: three by default; one in the register-lean instantiation)
                const int per_grp = (nparts + ngrp - 1) / ngrp;
                for (int k0 = 0; k0 < per_grp; k0 += MBATCH) {
                    f32x2 ml[MBATCH];
                    f32x2 t[MBATCH][NB][2];
#pragma unroll
                    for (int b = 0; b < MBATCH; ++b) {
                        const int sidx = min((member ? pg : 0) + ngrp * (k0 + b), nparts - 1);
                        const int64_t row = (int64_t)(first_run + sidx + seq) * p.Hq + hm;
                        ml[b] = load_dev2(p.part_ml + row * 2);
                        const float *ap = p.part_acc + row * HD + 4 * kq;
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb) {
                            t[b][nb][0] = load_dev2(ap + nb * 16);
                            t[b][nb][1] = load_dev2(ap + nb * 16 + 2);
                        }
                    }
#pragma unroll
                    for (int b = 0; b < MBATCH; ++b) {
                        if (member && pg + ngrp * (k0 + b) < nparts) {
                            f32x4 o2[NB];
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb)
                                o2[nb] = f32x4{t[b][nb][0][0], t[b][nb][0][1], t[b][nb][1][0], t[b][nb][1][1]};
                            fold(ml[b][0], ml[b][1], o2);
                        }
                    }
                }
                // groups 1 .. ngrp-1 into group 0 (lane col < g reads lane col + j*g of its 16-lane row);
                // a group that had no part carries (-inf, 0, 0) and changes nothing
                for (int j = 1; j < ngrp && j < nparts; ++j) {
                    const int src = (lane & ~15) | min(j * g + hc, 15);
                    const float m2 = __shfl(M, src), l2 = __shfl(ltot, src);
                    f32x4 o2[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int r = 0; r < 4; ++r) o2[nb][r] = __shfl(O[nb][r], src);
                    if (pg == 0) fold(m2, l2, o2);
                }
                if (lane == 0)   // ready for the next call
                    __hip_atomic_store(p.counters + (int64_t)seq * p.Hkv + kvh, 0, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                store_out = true;
            }
        }
        if (store_out && col < g) {
            const float inv = 1.0f / ltot;
            uint16_t *op = p.out + ((int64_t)q_row * p.Hq + head) * HD + 4 * kq;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                u32x2 w = {pack2_bf16(O[nb][0] * inv, O[nb][1] * inv), pack2_bf16(O[nb][2] * inv, O[nb][3] * inv)};
                *reinterpret_cast<u32x2 *>(op + nb * 16) = w;
            }
        }
        pos = stop;   // (the next piece's sequence is found at the top: ce <= pos unless the run ends here)
    }
}

// Entries of the decode array: lane l has entry l + 1 (for locate), and entry idx for the whole wave.  DEV: from device
// memory, where the plan did not fit the kernel arguments.
template <bool DEV>
OOCO_DEV int cum_head(const KernArgs &a, int lane)
{
    return DEV ? a.p.cum_dev[min(1 + lane, a.p.num_seqs)] : a.cum[1 + lane];
}
template <bool DEV>
OOCO_DEV int cum_entry(const KernArgs &a, int idx)
{
    return DEV ? a.p.cum_dev[idx] : a.cum[idx];
}

// GENERAL: XCD weights, a dynamic tail, or a plan in device memory (which equal runs without a tail may be, too).
template <int HD, int NBI, int MBATCH, bool GENERAL>
OOCO_DEV void decode_kernel_body(const KernArgs &a)
{
    const AttnParams &p = a.p;
    // What a wave needs before its first KV tile is on its way comes from a dozen places of the kernel
    // arguments; asked for one after the other, each at its point of use, they cost a wave ten dependent
    // round trips to the scalar cache.  Naming them here makes the compiler fetch them together.
    const int lane = threadIdx.x;
    asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.block_tables), "s"(p.seq_lens),
                 "s"(p.query_start_loc), "s"(p.cum_dev), "s"(p.trace), "s"(p.Hq), "s"(p.Hkv), "s"(p.g),
                 "s"(p.max_blocks_per_seq), "s"(p.num_seqs), "s"(p.total_q), "s"(p.dec_blocks), "s"(p.static_blocks),
                 "s"(p.static_runs), "s"(p.piece_pad), "s"((int)p.rotate_heads), "s"(p.scale_log2e));
    // Workgroups are handed to the XCDs round-robin and the kv heads of a block lie in adjacent
    // 4 KiB pieces of memory: rotating the head by the run index gives every XCD every kv head
    // in turn instead of pinning XCD x to head x.
    int run = blockIdx.x / p.Hkv;
    int kvh = p.rotate_heads ? (int)((blockIdx.x - run * p.Hkv + run) % p.Hkv) : (int)(blockIdx.x - run * p.Hkv);
    const bool dev = GENERAL && p.cum_dev;
    const int head = dev ? cum_head<true>(a, lane) : cum_head<false>(a, lane);
    auto cum_at = [&](int idx) -> int { return dev ? cum_entry<true>(a, idx) : cum_entry<false>(a, idx); };
    uint64_t *trace = p.trace ? p.trace + (int64_t)blockIdx.x * 4 : nullptr;   // per-wave time stamps
    if (trace && lane == 0) trace[0] = wall_clock64();
    bool first_piece = true;
    if constexpr (!GENERAL) {
        decode_run<HD, NBI, MBATCH>(p, cum_at, head, EqualRuns{p.static_blocks, p.static_runs}, run, kvh, lane, trace, first_piece, []() {});
    } else {
        if (p.xcd_cw[kXcds - 1]) {
            // weighted runs: all kv heads of run v on XCD v % 8 (workgroup b runs on XCD b % 8)
            const int x = blockIdx.x % kXcds, t = blockIdx.x / kXcds;
            kvh = t % p.Hkv;
            run = kXcds * (t / p.Hkv) + x;
        }
        const GeneralRuns L = {{p.dec_blocks, p.static_blocks, p.static_runs, p.tail_runs, p.xcd_cw}};
        const unsigned tail_tasks = (unsigned)p.tail_runs * (unsigned)p.Hkv;
        for (;;) {   // the wave's own run first, then tail runs by ticket
            // The ticket for the next tail run is drawn when the last piece of this run has been streamed (whoever
            // is done first gets the next run) and looked at after that piece's epilogue, which covers the round
            // trip of the atomic.  (Every wave ends by drawing a ticket that tells it to stop; atomics on one address
            // are served one after the other, about 13 ns each on MI355X, which is why the tail only pays on long
            // kernels.)
            unsigned ticket = 0xFFFFFFFFu;
            bool drawn = false;
            auto draw = [&]() {
                if (lane == 0)
                    ticket = __hip_atomic_fetch_add(p.queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - p.queue_base;
                drawn = true;
            };
            decode_run<HD, NBI, MBATCH>(p, cum_at, head, L, run, kvh, lane, trace, first_piece, [&]() {
                if (tail_tasks) draw();
            });
            if (!tail_tasks) break;
            if (!drawn) draw();   // (a run that held no block)
            ticket = __builtin_amdgcn_readfirstlane(ticket);
            if (ticket >= tail_tasks) break;
            run = p.static_runs + (int)(ticket / (unsigned)p.Hkv);
            kvh = (int)(ticket % (unsigned)p.Hkv);
        }
    }
    if (trace) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0) trace[3] = wall_clock64();
    }
}

template <int HD, int NBI>
__global__ __launch_bounds__(64, 2) void decode_kernel(const KernArgs a)
{
    decode_kernel_body<HD, NBI, 3, false>(a);
}
template <int HD, int NBI>
__global__ __launch_bounds__(64, 2) void decode_kernel_general(const KernArgs a)
{
    decode_kernel_body<HD, NBI, 3, true>(a);
}

// The same kernel within 160 registers per wave (one KV block per step, one part per merge round trip), for
// batches whose prefill workgroups need the rest of the register file: a SIMD then holds one decode wave beside
// two prefill waves of 176 registers.
template <int HD>
__global__ __launch_bounds__(64, 3) void decode_kernel_lean(const KernArgs a)
{
    decode_kernel_body<HD, 1, 1, false>(a);
}
template <int HD>
__global__ __launch_bounds__(64, 3) void decode_kernel_lean_general(const KernArgs a)
{
    decode_kernel_body<HD, 1, 1, true>(a);
}

// ------------------------------------------------------------------------------------------
// Cooperative decode: one workgroup of four waves per (run, kv head).  The waves share every piece of the run, step by
// step in turn, and merge their four results in LDS; only a piece that does not cover its whole sequence goes through
// the partial slots and the arrival counter, one part per workgroup, and the merge of those parts is done by all 256
// threads.  For small batches, whose time is the length of the chain
//   start -> steps of a wave, one after the other -> partial result -> arrival -> merge,
// this makes the chain short at both ends: a quarter of the steps per wave and of the parts per sequence.  Measured on
// MI355X against single waves: one sequence of 4000 tokens 14.1 -> 10.0 us, four of 60..200 (whole, nothing to merge
// through memory) 9.8 -> 5.1, sixteen of 2000..4000 (155 MB, then bound by HBM) 37.7 -> 36.2.
template <int HD>
constexpr int kCoopStride = HD + 16;   // floats from one head's partial output to the next in LDS (16-byte writes of four
                                       // heads' lanes then fall on 64 different banks)
template <int HD, int NWV>
constexpr int kCoopFloats = NWV * 16 * kCoopStride<HD> + NWV * 16 * 2 + 4;   // LDS the waves need

// (NWV = waves of the workgroup: 4, or 8 beside prefill workgroups of key groups)
// AHEAD = KV blocks that a wave's loads in flight belong to, those of the step at hand (V) and of the next (K): a step takes half
// of them, 8 KiB of tiles.  With steps of 16 KiB a wave has half as many, so the last of them is half empty more often, and the
// waves of a workgroup end further apart.  MI355X (us), steps of 16 -> 8 KiB: 24 decodes beside 237 rows, 28/4 heads 22.6 -> 20.1
// (148 workgroups of eight waves, 3.25 steps -> 6.5), four layers of 16 decodes 146.8 -> 138.7, 38 drawn batches 0.963 (0.885 ..
// 1.007); 4 KiB at head_dim 64 0.89 .. 1.11.
template <int HD, int AHEAD, int NWV, class CumAt>
OOCO_DEV void decode_coop_run(const AttnParams &p, CumAt cum_at, int cum_head, int run, int kvh, float *lds, uint64_t *trace)
{
    static_assert(AHEAD * HD == 256, "steps of 8 KiB");
    constexpr int NBI = AHEAD / 2;
    constexpr int NB = HD / 16;
    constexpr int STRIDE = kCoopStride<HD>;
    constexpr int THREADS = NWV * 64;
    constexpr int MAXU = (16 * HD / 4 + THREADS - 1) / THREADS;   // 16-byte units of the output a thread may own
    float *const l_ml = lds + NWV * 16 * STRIDE;
    int *const l_last = reinterpret_cast<int *>(l_ml + NWV * 16 * 2);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kq = lane >> 4;
    const int g = p.g, units = g * (HD / 4);
    bool first_piece = wave == 0;
    if (wave != 0) trace = nullptr;
    const EqualRuns L = {p.static_blocks, p.static_runs};
    int lo, hi, seq, cs, ce;
    if (p.coop == kCoopBySequence) {   // run i is sequence i, whole
        seq = run;
        cs = lo = cum_at(run);
        ce = hi = cum_at(run + 1);
        if (trace && lo >= hi && lane == 0) trace[1] = trace[2] = wall_clock64();
    } else {
        L.bounds(run, lo, hi);
        seq = locate(cum_at, cum_head, p.num_seqs, lo, lane, cs, ce);
    }
    int pos = lo;
    while (pos < hi) {   // (everything here is the same in all waves)
        while (ce <= pos) {   // the next sequence with decode blocks
            ++seq;
            cs = ce;
            ce = cum_at(seq + 1);
        }
        seq = __builtin_amdgcn_readfirstlane(seq);
        const int stop = min(hi, ce);
        const int first = cs + p.piece_pad;
        const int begin = max(pos, first);
        if (begin >= stop) {   // the run ends before the first block of this sequence
            if (trace && lane == 0) trace[2] = wall_clock64();
            pos = stop;
            continue;
        }
        const bool whole = (begin == first) && (stop == ce);
        f32x4 O[NB];
        float m, lsum;
        int q_row;
        decode_stream<HD, NBI, NWV>(p, kvh, seq, begin - first, stop - begin, q_row, wave, lane, trace, first_piece, O, m, lsum);
        if (trace && stop == hi && lane == 0) trace[2] = wall_clock64();
        const float lw = rows_sum(lsum);
        if (pos != lo) __syncthreads();   // the last piece's results have been read
        if (col < g) {
            float *o = lds + (wave * 16 + col) * STRIDE + 4 * kq;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) *reinterpret_cast<f32x4 *>(o + 16 * nb) = O[nb];
            if (kq == 0) *reinterpret_cast<f32x2 *>(l_ml + (wave * 16 + col) * 2) = f32x2{m, lw};
        }
        __syncthreads();
        auto put = [&](int hh, int d4, const f32x4 &acc, float l) {
            const float inv = 1.0f / l;
            uint16_t *op = p.out + ((int64_t)q_row * p.Hq + kvh * g + hh) * HD + 4 * d4;
            *reinterpret_cast<u32x2 *>(op) = u32x2{pack2_bf16(acc[0] * inv, acc[1] * inv), pack2_bf16(acc[2] * inv, acc[3] * inv)};
        };
#pragma unroll
        for (int i = 0; i < MAXU; ++i) {
            const int u = tid + THREADS * i;
            if (u < units) {
                const int hh = u / (HD / 4), d4 = u % (HD / 4);
                f32x2 ml[NWV];
#pragma unroll
                for (int w = 0; w < NWV; ++w) ml[w] = *reinterpret_cast<const f32x2 *>(l_ml + (w * 16 + hh) * 2);
                float M = ml[0][0];
#pragma unroll
                for (int w = 1; w < NWV; ++w) M = fmaxf(M, ml[w][0]);
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                float l = 0.f;
#pragma unroll
                for (int w = 0; w < NWV; ++w) {   // in wave order
                    const float wt = fast_exp2(ml[w][0] - M);
                    const f32x4 o = *reinterpret_cast<const f32x4 *>(lds + (w * 16 + hh) * STRIDE + 4 * d4);
                    l += ml[w][1] * wt;
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[r] += o[r] * wt;
                }
                if (whole) {
                    put(hh, d4, acc, l);
                } else {
                    const int64_t row = (int64_t)(run + seq) * p.Hq + kvh * g + hh;
                    store_dev4(p.part_acc + row * HD + 4 * d4, acc);
                    if (d4 == 0) store_dev2(p.part_ml + row * 2, M, l);
                }
            }
        }
        if (!whole) {
            int first_run, last_run;
            L.holding(first, ce - 1, first_run, last_run);
            const int nparts = last_run - first_run + 1;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partial has reached memory ...
            __syncthreads();                                    // ... and so have the other waves'
            int32_t *const counter = p.counters + (int64_t)seq * p.Hkv + kvh;
            if (tid == 0) *l_last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nparts - 1;
            __syncthreads();
            if (*l_last) {   // last part of this (sequence, kv head): merge, in slot order
#pragma unroll
                for (int i = 0; i < MAXU; ++i) {
                    const int u = tid + THREADS * i;
                    if (u < units) {
                        const int hh = u / (HD / 4), d4 = u % (HD / 4);
                        float M = -INFINITY, l = 0.f;
                        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                        auto merge = [&](auto batch, int j0) {   // parts j0 .. whose loads are on their way together
                            constexpr int BATCH = decltype(batch)::value;
                            f32x2 ml[BATCH], t[BATCH][2];
#pragma unroll
                            for (int b = 0; b < BATCH; ++b) {
                                const int64_t row = (int64_t)(first_run + min(j0 + b, nparts - 1) + seq) * p.Hq + kvh * g + hh;
                                ml[b] = load_dev2(p.part_ml + row * 2);
                                t[b][0] = load_dev2(p.part_acc + row * HD + 4 * d4);
                                t[b][1] = load_dev2(p.part_acc + row * HD + 4 * d4 + 2);
                            }
#pragma unroll
                            for (int b = 0; b < BATCH; ++b) {
                                if (j0 + b < nparts) {
                                    const float M_new = fmaxf(M, ml[b][0]);
                                    const float w_old = fast_exp2(M - M_new), w_new = fast_exp2(ml[b][0] - M_new);
                                    M = M_new;
                                    l = l * w_old + ml[b][1] * w_new;
#pragma unroll
                                    for (int r = 0; r < 4; ++r) acc[r] = acc[r] * w_old + t[b][r >> 1][r & 1] * w_new;
                                }
                            }
                        };
                        int j0 = 0;
                        for (; j0 + 4 < nparts; j0 += 16) merge(std::integral_constant<int, 16>(), j0);
                        if (j0 < nparts) merge(std::integral_constant<int, 4>(), j0);
                        put(hh, d4, acc, l);
                    }
                }
                if (tid == 0)   // ready for the next call
                    __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        pos = stop;
    }
}

template <int HD, int AHEAD, int NWV, bool DEV>
OOCO_DEV void decode_coop_kernel_body(const KernArgs &a)
{
    const AttnParams &p = a.p;
    __shared__ __align__(16) float lds[kCoopFloats<HD, NWV>];
    asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.block_tables), "s"(p.seq_lens), "s"(p.query_start_loc),
                 "s"(p.cum_dev), "s"(p.trace), "s"(p.Hq), "s"(p.Hkv), "s"(p.g), "s"(p.max_blocks_per_seq), "s"(p.num_seqs),
                 "s"(p.total_q), "s"(p.dec_blocks), "s"(p.static_blocks), "s"(p.static_runs), "s"(p.piece_pad),
                 "s"((int)p.rotate_heads), "s"(p.scale_log2e));
    const int run = blockIdx.x / p.Hkv, slot = blockIdx.x - run * p.Hkv;
    const int kvh = p.rotate_heads ? (slot + run) % p.Hkv : slot;
    uint64_t *const trace = p.trace ? p.trace + (int64_t)blockIdx.x * 4 : nullptr;
    if (trace && threadIdx.x == 0) trace[0] = wall_clock64();
    decode_coop_run<HD, AHEAD, NWV>(p, [&](int idx) -> int { return cum_entry<DEV>(a, idx); }, cum_head<DEV>(a, threadIdx.x & 63), run, kvh,
                                  lds, trace);
    if (trace) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (threadIdx.x == 0) trace[3] = wall_clock64();
    }
}
template <int HD, int AHEAD>
__global__ __launch_bounds__(256, 2) void decode_coop_kernel(const KernArgs a)
{
    decode_coop_kernel_body<HD, AHEAD, 4, false>(a);
}
template <int HD, int AHEAD>
__global__ __launch_bounds__(256, 2) void decode_coop_kernel_general(const KernArgs a)   // a plan in device memory
{
    decode_coop_kernel_body<HD, AHEAD, 4, true>(a);
}
template <int HD, int AHEAD>
__global__ __launch_bounds__(512, 2) void decode_coop_kernel_groups(const KernArgs a)   // eight waves, beside key groups
{
    decode_coop_kernel_body<HD, AHEAD, 8, false>(a);
}

// ------------------------------------------------------------------------------------------
// Prefill chunk: one workgroup of four waves per (tile of query rows, kv head).  The 128 query
// columns of a workgroup are the (row, head) pairs of tile_rows = 128/g consecutive query rows
// and the g query heads that share the kv head (column c = row*g + head), 32 columns per wave,
// so every K/V tile fetched serves the whole GQA group.  KV is walked four blocks (64 tokens) per
// step through two LDS slots for K and two for V (64 KiB for hd 128), filled by direct
// global->LDS loads, one barrier per step.  Per wave and step, for each 32-token half:
//   S^T[32 tok][32 cols] = K · Q^T    (hd/16 x v_mfma_f32_32x32x16_bf16, K operand from LDS)
//   O^T[hd][32 cols]    += V^T · P^T  (hd/32 x 2 x v_mfma_f32_32x32x16_bf16, V operand from LDS)
// The loop is software pipelined over halves of 32 tokens: a region of 16 MFMAs multiplies the weights of one half by V and
// computes the scores of a half two further on, while the vector ALU turns the scores of the half between them into weights,
// a score or so per MFMA.  K therefore runs one step ahead of V: in step st the loads of K[st+2] and V[st+1] are sent off.
// Lane l = 32*h + col.  MFMA row i of the K operand is fed with token (i with bits 2 and 3
// swapped) of its block, so that S^T register r of lane (col, h) is token 16(r/8) + 8h + r%8 of
// the half: eight consecutive tokens per block, which is what one 16-byte V operand holds.
// LDS (16-byte units, CH = 2*hd per tile): K tiles keep the cache order [hd/8][16 slots]; V tiles
// are stored [token half][dim] so that the 16 lanes of a quarter wave read 256 contiguous bytes
// (no bank conflicts).
// What bounds it, by stamps of the clock counter and loops of the same instruction mix on their own (cycles per 32x32x16 MFMA,
// which takes 32, of two waves on a SIMD): on zeros the issue of everything around the matrix cores, on random data the power
// that they draw, which brings the clock from 2.4 to 1.6 .. 1.75 GHz.  Both ask for few instructions per MFMA, at even distances:
//   * an exponential, its fma and half a conversion per MFMA run beside it (67 cycles per pair of MFMAs); v_dot2c_f32_bf16 does
//     not (84), so the sums of the weights are a small matrix product (73);
//   * no maximum: weights are computed against the reference as it stands, and their sums show when it has to move;
//   * the loads of a step are issued between MFMAs: all at its start they took a wave 860 of 3500 cycles; a wave's pieces lie in
//     one block, so that a step asks it for one block id, two tile addresses and two settings of M0;
//   * the barrier of a step sits where the last operands of the step before it are on their way to registers.
// MI355X (us, before -> after): 2 x 2048 rows on 4096 tokens, 64/8 heads 602 -> 574 (on zeros 448 -> 400), 8 x 512 rows on up to
// 2048, 32/8 heads 85.7 -> 81.1, 300 rows on 14,683 tokens 87.0 -> 82.5.  (Calls as a whole, with the output stores and the
// operands below as well: 608 -> 576, 89.3 -> 78.5, 256 rows on 8192 tokens 86.6 -> 81.5.)
// The causal mask runs only on halves that touch the diagonal; at the end of a sequence the unused V slots are zeroed once in LDS
// instead of masking operands.  Two workgroups fit a CU (<= 256 VGPRs, 64 KiB LDS each), three of head_dim 64 (<= 168, 32 KiB).
constexpr int kPfThreads = 256;   // threads of the four-wave workgroup (the eight-wave one has 512)
constexpr int kPfBlocks = 4;    // KV blocks per step
constexpr int kSharedMergeParts = 4;   // parts from which sharing the merge of a split tile pays (see prefill_unit)

// Entry idx of the plan's array: from device memory if the plan did not fit the kernel arguments, else from the
// argument block.  The two loads must stay two loads: merged into one load through a selected pointer, the argument
// block would have to be addressable like memory, and the compiler would copy all 4 KiB of it into every lane's
// private memory (the empty asm keeps the arms of the branch apart).
OOCO_DEV int plan_entry(const KernArgs &a, int idx)
{
    if (a.p.cum_dev) return a.p.cum_dev[idx];
    int v = a.cum[idx];
    asm volatile("" : "+v"(v));
    return v;
}

// The K and V tiles of two steps, for KG key groups, as one array (the cooperative decode workgroups of the step kernel use
// the same memory).
template <int KG>
constexpr int kPfGroupBlocks = KG == 1 ? kPfBlocks : 2 * kPfBlocks / KG;   // KV blocks a key group stages per step
template <int HD, int KG = 1>
OOCO_DEV u32x4 *stage_lds()
{
    __shared__ u32x4 lds[4 * KG * kPfGroupBlocks<KG> * HD * 2];
    return lds;
}

// One workgroup's work on virtual block index `vb` (what blockIdx.x is in the stand-alone kernel): with the plan's
// tile list, entry vb / Hkv of the list -- a (tile, part of its keys) pair -- for kv head vb % Hkv; without it, unit
// vb / split = (tile, kv head), part vb % split of its keys.  `cum_at(i)` reads the prefill array of the plan.  All
// threads of the workgroup call it together; every return is workgroup-uniform.
// NW = waves per workgroup: 4 (128 query columns) or 8 (256 columns: the same K/V tiles in LDS serve twice as many
// columns, which halves the traffic from L2 into the compute unit per unit of matrix work).
// KG = key groups: with 4, the NW = 8 waves are four groups of two, 64 query columns, and each group stages and walks a
// quarter (32) of every 128 keys with a pipeline of its own; only the barrier of a step is common.  The groups' results meet
// in LDS (128 KiB, as much as their tiles: one workgroup per compute unit).  For batches of few tiles, which are bound by
// the chain of steps and not by the matrix cores: a step takes about the time its loads need whatever it holds (1.06 .. 1.36 us
// for 128 keys in place of 1.08 .. 1.3 for 64 when the rule was measured; both became 5 to 12 % shorter since), and a tile of few columns keeps a quarter of the waves idle instead of
// three quarters.  Measured on MI355X against KG = 1 (us): 3 chunks of 3 rows on 17,000 cached tokens, 28/4 heads 42.6 -> 28.3,
// 57 + 87 rows on 2000, 32/8 20.7 -> 18.0, 3 x 100 rows on 400 15.5 -> 12.5; two groups of 128 columns each gained nothing
// (1 x 300 rows on 15,780 tokens 93.9 against 93.7, short contexts 2.5 us for the merge of 128 KiB).
// PIPE = false: no software pipeline across steps (the scores of a step are computed in that step, one score
// register set): fewer registers, so that two such waves and a decode wave share a SIMD; the overlap of matrix and
// vector work then comes from the two waves of a SIMD rather than from within one wave.
// `phases` (option "trace", prefill-only batches): receives four 16-bit times in units of 10 ns since `t_start`
// (saturating), lowest first: tile looked up, first K/V loads sent off, first tiles arrived, last step done.
// `list_word`: with the tile list, the word of the workgroup's entry vb / Hkv.
template <int HD, int NW, bool PIPE, int KG, class CumAt>
OOCO_DEV void prefill_unit(const AttnParams &p, CumAt cum_at, const int vb, const int entry, const int list_kvh, const int list_word,
                           uint64_t *phases = nullptr, const uint64_t t_start = 0)
{
    constexpr int NC = NW / KG;        // waves per key group, 32 query columns each
    constexpr int COLS = NC * 32;      // query columns per workgroup
    constexpr int KS = HD / 16;        // k-steps of QK
    constexpr int MB = HD / 32;        // 32-dim groups of the output
    constexpr int CH = HD * 2;         // 16-byte chunks per (block, kv head) tile
    constexpr int BLK = kPfGroupBlocks<KG>;             // KV blocks of one step of a key group
    constexpr int T = BLK * kBlockSize, HV = T / 32;    // tokens, and 32-token halves, of such a step
    constexpr int STEP = KG * T;                        // tokens of one step of the workgroup
    constexpr int STAGE = BLK * CH;                     // chunks of one step's K (or V) tiles of a key group
    constexpr int NCP = STAGE / (NC * 64);              // chunks each thread moves per stage
    constexpr int ITEMS = 4 * MB / KG;                  // 16-byte pieces of the merged output a thread ends up with

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = KG == 1 ? 0 : wave_id / NC, wave = KG == 1 ? wave_id : wave_id - kg * NC;   // key group, wave of the group
    u32x4 (*const ldsK)[STAGE] = reinterpret_cast<u32x4 (*)[STAGE]>(stage_lds<HD, KG>()) + 4 * kg, (*const ldsV)[STAGE] = ldsK + 2;
    const int col = lane & 31;
    const int h = lane >> 5;
    const int g = p.g;
    uint64_t phase_bits = 0;   // (scalar; touched only when tracing)
    auto phase = [&](int k) {
        if (phases) {
            const uint64_t dt = (uint64_t)wall_clock64() - t_start;
            phase_bits |= (dt < 0xFFFFu ? dt : (uint64_t)0xFFFFu) << (16 * k);
        }
    };
    // workgroup -> (tile, kv head, part of the tile's keys, parts the tile has), and the partial-result slot of
    // part 0 of that (tile, kv head) with the distance between the slots of consecutive parts.  With the tile list
    // every tile has its own number of parts; without it vb = ((tile * Hkv) + kv head) * pf_split + part.
    int split, part, kvh, seq, t;
    int slot0, slot_step;   // (at most kPrefillSplitUnits * kMaxPrefillSplit slots)
    if (p.pf_table) {   // the plan lists the (tile, part) pairs one by one
        const int list_e = __builtin_amdgcn_readfirstlane(list_word);   // (the same in every lane)
        kvh = __builtin_amdgcn_readfirstlane(list_kvh);
        part = entry_part(list_e);
        split = entry_parts(list_e);
        slot0 = (entry - part) * p.Hkv + kvh;
        slot_step = p.Hkv;
        t = entry_tile(list_e);
        seq = p.list_by_seq ? entry_chunk(list_e) : cum_at(p.num_pf + 1 + min(entry_chunk(list_e), p.num_pf - 1));
    } else {
        split = p.pf_split;
        const int unit = vb / split;
        part = __builtin_amdgcn_readfirstlane(vb - unit * split);
        const int tile_idx = unit / p.Hkv;
        kvh = __builtin_amdgcn_readfirstlane(unit - tile_idx * p.Hkv);
        slot0 = unit * split;
        slot_step = 1;
        // tile -> (sequence, tile of the sequence); tiles of a sequence are taken last-first because
        // the later rows of a chunk see more keys and the hardware dispatches in index order
        const int chunk = __builtin_amdgcn_readfirstlane(count_le(cum_at, p.num_pf, tile_idx, lane));
        t = __builtin_amdgcn_readfirstlane((cum_at(chunk + 1) - 1) - tile_idx);   // reversed order inside the sequence
        seq = cum_at(p.num_pf + 1 + chunk);
    }
    seq = __builtin_amdgcn_readfirstlane(min(max(seq, 0), p.num_seqs - 1));
    // The sequence's lengths, and the block ids of the first three steps where the workgroup starts at the first key, in one
    // round trip (through the constant address space: scalar loads, which the waits on the vector-memory counter do not see).
    // Ids past the tile's last block may be anything until they are replaced below.
    typedef const __attribute__((address_space(4))) int32_t *const_i32_ptr;
    const const_i32_ptr ctable = (const_i32_ptr)(uintptr_t)(p.block_tables + (int64_t)seq * p.max_blocks_per_seq);
    // A wave moves NCP consecutive 64-chunk pieces of a stage, which lie in one block: the first is chunk piece_chunk of block
    // piece_block of the step.  (APART: the wave's two pieces are the same quarter of two blocks, two apart; see issue.)
    constexpr bool APART = !PIPE;
    const int piece_block = APART ? wave >> 2 : wave * NCP * 64 / CH, piece_chunk = APART ? (wave & 3) * 64 : wave * NCP * 64 % CH;
    static_assert(CH % (NCP * 64) == 0 && (!APART || (NC == 8 && CH == 256)), "where the pieces of a wave lie");
    auto wave_block = [&](int st) -> int { return BLK * (KG * st + kg) + piece_block; };   // of the sequence
    int id0, id1, id2;   // physical ids of this wave's blocks of the steps st, st + 1 and st + 2
    int id0b, id1b;      // (APART: of the second blocks of the steps st and st + 1)
    const int id_first = ctable[0];
    {
        const int last = p.max_blocks_per_seq - 1;
        id0 = ctable[min(wave_block(0), last)];
        id1 = ctable[min(wave_block(1), last)];
        id2 = ctable[min(wave_block(2), last)];
        if constexpr (APART) {
            id0b = ctable[min(wave_block(0) + 2, last)];
            id1b = ctable[min(wave_block(1) + 2, last)];
        }
    }
    int q_row0, rows, pos0, seq_len;
    {
        const const_i32_ptr qsl = (const_i32_ptr)(uintptr_t)p.query_start_loc;
        const int q0 = qsl[seq], q1 = qsl[seq + 1];
        const int ctx = ((const_i32_ptr)(uintptr_t)p.ctx_lens)[seq];
        seq_len = ((const_i32_ptr)(uintptr_t)p.seq_lens)[seq];
        const int q_len = q1 - q0;
        const int tile_rows = max(1, (COLS * (int)p.g_magic) >> 15);
        const int t0 = t * tile_rows;
        q_row0 = min(max(q0 + t0, 0), p.total_q - 1);
        rows = max(1, min(min(tile_rows, q_len - t0), p.total_q - q_row0));
        // keys beyond what the plan allotted to this sequence are never touched
        const int cap = p.max_blocks_per_seq * kBlockSize;
        pos0 = min(max(ctx + t0, 0), cap - rows);
        seq_len = min(seq_len, cap);
    }
    const uint16_t *const k_cache = p.k_cache, *const v_cache = p.v_cache;
    const int Hkv = p.Hkv;
    const float c_log2e = p.scale_log2e;
    const uint32_t ldsK_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)&ldsK[0][0];
    const uint32_t ldsV_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)&ldsV[0][0];
    // this lane's query column
    const int c = wave * 32 + col;
    const int c_row = (int)((uint32_t)c * p.g_magic >> 15), c_head = c - c_row * g;
    const int row = min(c_row, rows - 1);
    const int head = kvh * g + c_head;
    const int pos = pos0 + row;                          // this column's absolute position
    // the wave's columns span rows [w_row_lo, w_row_hi] (scalar)
    const int w_row_lo = min((wave * 32 * (int)p.g_magic) >> 15, rows - 1), w_row_hi = min(((wave * 32 + 31) * (int)p.g_magic) >> 15, rows - 1);
    const bool w_used = wave * 32 < rows * g;            // (a narrow tile leaves the other waves without columns: they only stage)
    const int w_pos_lo = pos0 + w_row_lo, w_pos_hi = w_used ? pos0 + w_row_hi : -1;
    const int kv_end = pos0 + rows;                      // keys visible to the tile: [0, kv_end)
    const int nblk = (kv_end + kBlockSize - 1) / kBlockSize;
    const int nstep_all = (nblk + KG * BLK - 1) / (KG * BLK);
    // this workgroup's share of the steps: [st_lo, nstep); a unit with fewer steps than parts has fewer parts
    const int nparts = min(split, nstep_all);
    if (part >= nparts) return;                          // (the whole workgroup leaves: no barrier is pending)
    const int st_lo = nstep_all * part / nparts;
    const int nstep = nstep_all * (part + 1) / nparts;

    phase(0);
    u32x4 qb[KS];
    {
        const u32x4 *qp = reinterpret_cast<const u32x4 *>(p.q + ((int64_t)(q_row0 + row) * p.Hq + head) * HD);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qb[ks] = qp[2 * ks + h];
    }
    const int64_t tile_elems = (int64_t)HD * kBlockSize;
    // K operand row col -> block (col>>4) of the half, slot with bits 2,3 of (col&15) swapped
    const int ku = col >> 4;
    const int kslot = (col & 3) | ((col & 4) << 1) | ((col & 8) >> 1);

    // One stage (the K or the V tiles of a step) goes from global memory straight into LDS (global_load_lds_dwordx4: every lane
    // gives a 16-byte global address, the wave's 64 pieces land contiguously at the LDS address in M0; the instruction's offset
    // counts for both).  Chunk c of a block's tile in LDS comes from
    //   K: cache chunk c   (same order as the cache)
    //   V: half = c / HD, dim = c % HD  <-  cache chunk 2*dim + half
    // The instructions are issued through inline asm so that the waits stay under this code's control.
    const uint32_t blk_bytes = (uint32_t)Hkv * (uint32_t)tile_elems * 2u;
    constexpr int kBias = 2048;   // keeps the V offsets below positive
    const char *const k_head = reinterpret_cast<const char *>(k_cache + (int64_t)kvh * tile_elems);
    const char *const v_head = reinterpret_cast<const char *>(v_cache + (int64_t)kvh * tile_elems) - kBias;
    const uint32_t k_off = (uint32_t)(piece_chunk + lane) * 16u;
    uint32_t v_off[NCP];
#pragma unroll
    for (int n = 0; n < NCP; ++n) {
        const int c = piece_chunk + (APART ? 0 : n * 64) + lane;
        v_off[n] = (uint32_t)((2 * (c % HD) + c / HD) * 16 - (APART ? 0 : n * 1024) + kBias);
    }
    // all pieces of this wave, of block id (scalar tile address + 32-bit lane offset)
    auto issue = [&](bool is_v, int slot, int id) {
        const char *const base = (is_v ? v_head : k_head) + (uint64_t)(uint32_t)id * blk_bytes;
        const uint32_t dst = (is_v ? ldsV_base : ldsK_base) + (uint32_t)((slot * STAGE + wave * NCP * 64) * 16);
        uint32_t off[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) off[n] = is_v ? v_off[n % NCP] : k_off;
        uint32_t saved_m0;   // M0 is restored: the compiler may keep a value of its own there
        if constexpr (NCP == 4)
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                         "global_load_lds_dwordx4 %2, %6\n\tglobal_load_lds_dwordx4 %3, %6 offset:1024\n\t"
                         "global_load_lds_dwordx4 %4, %6 offset:2048\n\tglobal_load_lds_dwordx4 %5, %6 offset:3072\n\ts_mov_b32 m0, %0"
                         : "=&s"(saved_m0)
                         : "s"(dst), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base)
                         : "memory");
        else
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                         "global_load_lds_dwordx4 %2, %4\n\tglobal_load_lds_dwordx4 %3, %4 offset:1024\n\ts_mov_b32 m0, %0"
                         : "=&s"(saved_m0)
                         : "s"(dst), "v"(off[0]), "v"(off[1]), "s"(base)
                         : "memory");
        static_assert(NCP == 2 || NCP == 4, "one asm statement");
    };
    // With eight waves and no pipeline, beside decode waves, the quarters of a block are fetched by four waves side by side, one load
    // from each of two blocks, as fast as a wave can: two pieces of one block per wave cost the decode stream 0.8 % (MI355X, 2 x
    // 2048 rows and 32 long decodes 1648 -> 1659 us, 8 x 512 and 128 262.6 -> 265.3).
    auto issue_apart = [&](bool is_v, int slot, int ida, int idb) {
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const char *const base = (is_v ? v_head : k_head) + (uint64_t)(uint32_t)(n ? idb : ida) * blk_bytes;
            const uint32_t dst = (is_v ? ldsV_base : ldsK_base) + (uint32_t)((slot * STAGE + (2 * n + piece_block) * CH + piece_chunk) * 16);
            const uint32_t off = is_v ? v_off[0] : k_off;
            uint32_t saved_m0;
            asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                         : "=&s"(saved_m0)
                         : "s"(dst), "v"(off), "s"(base)
                         : "memory");
        }
    };
    f32x16 O[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[mb][r] = 0.f;

    // scores of 32 tokens: S register r is token 8h + 16(r/8) + r%8 of them
    float m = -1e30f;   // (finite, so that a half of which a column sees nothing gives it weights of 0 and not inf - inf)
    // The sums of the weights come from the matrix cores too (v_mfma_f32_16x16x32_bf16): as an operand of that product the 16
    // rounded weights of a lane pair are 16 columns by 32 rows, of which rows 0..7 and 16..23 belong to columns 0..15 of the wave
    // and the others to columns 16..31, so a first operand of ones and zeros gives both sums, in every lane those of columns
    // lane % 16 and 16 + lane % 16.  (v_dot2c_f32_bf16 does not run beside matrix instructions: two waves per SIMD of MFMA + LDS
    // read + a score's exponential 84 cycles per pair of MFMAs with it, 73 with this product, 67 without any sum.)
    u32x4 ones;
#pragma unroll
    for (int w = 0; w < 4; ++w) ones[w] = ((lane >> 4) & 1) == (lane & 1) ? 0x3F803F80u : 0u;
    auto add_weights = [&](const u32x4 &P, f32x4 &sums) {
        sums = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ones), __builtin_bit_cast(bf16x8, P), sums, 0, 0, 0);
    };
    // Weights are computed against the reference m as it stands.  It only has to keep them in range (the final division cancels
    // it, weights above 1 are as exact in bf16 and fp32 as below), so it moves when the weights of a column's half step sum to
    // more than kMaxWeights, or to infinity or NaN, and then the half is done again (move_reference).
    constexpr float kMaxWeights = 256.0f, kMargin = 8.0f;
    auto weights16 = [&](const f32x16 &S, u32x4 (&P)[2], f32x4 &sums) {
        sums = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float e[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) e[r] = fast_exp2(__builtin_fmaf(S[8 * q + r], c_log2e, -m));
            P[q] = u32x4{pack2_bf16(e[0], e[1]), pack2_bf16(e[2], e[3]), pack2_bf16(e[4], e[5]), pack2_bf16(e[6], e[7])};
            add_weights(P[q], sums);
        }
    };
    auto too_large = [&](const f32x4 &sums) -> bool { return !__all(sums[0] <= kMaxWeights && sums[1] <= kMaxWeights); };   // (or NaN)
    float lsum_lo = 0.f, lsum_hi = 0.f;   // running sums of columns lane % 16 and 16 + lane % 16
    auto mask16 = [&](f32x16 &S, int tok0) {   // tok0: first token of the 32
        const int room = pos - (tok0 + 8 * h);
#pragma unroll
        for (int r = 0; r < 16; ++r) S[r] = (16 * (r / 8) + (r % 8) <= room) ? S[r] : -INFINITY;
    };
    // Last step of a sequence only (workgroup-uniform): V slots at or past seq_len may hold anything; their
    // weights are 0, but 0*NaN is NaN, so they are zeroed in LDS before anybody multiplies with them.
    auto scrub_v = [&](int slot, int tok0) {
#pragma unroll
        for (int n = 0; n < NCP; ++n) {
            const int cidx = (n * NC + wave) * 64 + lane;    // chunk [block][token half][dim] of the stage
            const int blk = cidx / CH, half = (cidx % CH) / HD;
            const int t0 = tok0 + 16 * blk + 8 * half;       // tokens t0 .. t0+7
            u32x4 mk;
#pragma unroll
            for (int w = 0; w < 4; ++w)
                mk[w] = (t0 + 2 * w < seq_len ? 0x0000FFFFu : 0u) | (t0 + 2 * w + 1 < seq_len ? 0xFFFF0000u : 0u);
            ldsV[slot][cidx] &= mk;
        }
        __syncthreads();
    };

    // Block ids of further steps: lane l holds this wave's block of step id_base + l, and of step id_base + 64 + l.
    const int32_t *const vtable = p.block_tables + (int64_t)seq * p.max_blocks_per_seq;
    int id_base = st_lo + 3, idv = 0, idn = 0;
    auto next_id = [&](int st) -> int {   // st is wave-uniform and does not decrease
        if (st - id_base >= 64) {
            id_base += 64;
            idv = idn;
            asm volatile("" : "+v"(idv));   // (waited for here, in the rare path)
            idn = vtable[min(wave_block(id_base + 64 + lane), nblk - 1)];
        }
        return __builtin_amdgcn_readlane(idv, st - id_base);
    };
    {
        if (st_lo == 0) {   // (the ids are here; steps past the tile's last block take any valid one)
            if (wave_block(0) >= nblk) id0 = id_first;
            if (wave_block(1) >= nblk) id1 = id_first;
            if (wave_block(2) >= nblk) id2 = id_first;
            if constexpr (APART) {
                if (wave_block(0) + 2 >= nblk) id0b = id_first;
                if (wave_block(1) + 2 >= nblk) id1b = id_first;
            }
        } else {
            id0 = ctable[min(wave_block(st_lo), nblk - 1)];
            id1 = ctable[min(wave_block(st_lo + 1), nblk - 1)];
            id2 = ctable[min(wave_block(st_lo + 2), nblk - 1)];
            if constexpr (APART) {
                id0b = ctable[min(wave_block(st_lo) + 2, nblk - 1)];
                id1b = ctable[min(wave_block(st_lo + 1) + 2, nblk - 1)];
            }
        }
        if constexpr (APART) {
            issue_apart(false, st_lo & 1, id0, id0b);
            issue_apart(true, st_lo & 1, id0, id0b);
        } else {
            issue(false, st_lo & 1, id0);
            issue(true, st_lo & 1, id0);
            if (st_lo + 1 < nstep) issue(false, (st_lo + 1) & 1, id1);
        }
        if constexpr (PIPE) {
            idv = vtable[min(wave_block(id_base + lane), nblk - 1)];
            idn = vtable[min(wave_block(id_base + 64 + lane), nblk - 1)];
        }
        // Passing the query registers through an empty asm makes the compiler wait for their loads here, behind the first
        // tiles' loads and before the loop, instead of counting them down inside it (which would also wait for the
        // global->LDS loads it does not know about).
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qb[ks]));
    }
    phase(1);
    // A region: the weights Pu of 32 tokens by V (PV), the scores Ss of 32 others turned into the weights Pn (NEXT), and the scores
    // Sq of 32 more (QK), hd/16 MFMAs for each of the two products, in turn, with the vector work spread evenly between them.
    // Every LDS operand is asked for AHEAD MFMAs before its own, the first of a region by the region before it.  Two are enough, and
    // hold fewer registers: at head_dim 64 a SIMD then has three waves (158 registers for 172).  MI355X (us), four -> two: 2 x 2048 rows
    // on 4096 tokens, 64/8 heads 580.6 -> 576.0, 4 chunks of 700..1100, 28/4 heads 95.9 -> 93.6; head_dim 64: 8 x 450 rows 43.8 -> 42.4,
    // ten drawn batches 0.97; key groups of head_dim 128, 2 x 133 rows on 1231 tokens 16.8 -> 16.9.
    constexpr int AHEAD = KG > 1 && HD == 128 ? 4 : 2;
    u32x4 ring[AHEAD];
    auto operand = [&](auto pv, auto qk, int i, int vslot, int vhalf, int kslot_q, int khalf) -> u32x4 {   // of MFMA i of a region
        constexpr bool PV = decltype(pv)::value, QK = decltype(qk)::value;
        const int j = PV && QK ? i / 2 : i;
        if (QK && (!PV || (i & 1) == 0)) return ldsK[kslot_q][(2 * khalf + ku) * CH + h * 16 + kslot + j * 32];
        return ldsV[vslot][(2 * vhalf + j / MB) * CH + h * HD + col + 32 * (j % MB)];
    };
    // prefetch(i): asks for operand i of the next region; beside(i): called once MFMA i has been issued
    auto region = [&](auto pv, auto qk, auto next, u32x4 (&Pu)[2], f32x4 &sums_u, int vslot, int vhalf, f32x16 &Ss, u32x4 (&Pn)[2],
                      f32x4 &sums_n, f32x16 &Sq, int kslot_q, int khalf, auto &&prefetch, auto &&beside) {
        constexpr bool PV = decltype(pv)::value, QK = decltype(qk)::value, NEXT = decltype(next)::value;
        constexpr int NM = (PV ? KS : 0) + (QK ? KS : 0);
        static_assert(2 * MB == KS, "as many products of each kind");
        if constexpr (PV) {
            lsum_lo += sums_u[0];
            lsum_hi += sums_u[1];
        }
        float e[16];
        f32x4 sums = {0.f, 0.f, 0.f, 0.f};
        // the vector work of score r, one stage later per two scores: scaled and referenced, exponentiated, packed and summed
        auto vector_work = [&](int r) {
            if (r < 16) e[r] = __builtin_fmaf(Ss[r], c_log2e, -m);
            const int x = r - 2;
            if (x >= 0 && x < 16) e[x] = fast_exp2(e[x]);
            const int y = r - 4;
            if (y >= 0 && y < 16 && (y & 1)) {
                Pn[y / 8][(y % 8) / 2] = pack2_bf16(e[y - 1], e[y]);
                if (y % 8 == 7) add_weights(Pn[y / 8], sums);
            }
        };
        constexpr int CALLS = 20, OVER = NM - 2;   // calls of vector_work for 16 scores, MFMAs that they are spread over
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int j = PV && QK ? i / 2 : i;
            const u32x4 op = ring[i % AHEAD];
            if (QK && (!PV || (i & 1) == 0)) {
                f32x16 z;
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = 0.f;
                Sq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op), __builtin_bit_cast(bf16x8, qb[j]),
                                                             j == 0 ? z : Sq, 0, 0, 0);
            } else {
                O[j % MB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, op), __builtin_bit_cast(bf16x8, Pu[j / MB]),
                                                                    O[j % MB], 0, 0, 0);
            }
            beside(i);
            if (i + AHEAD < NM)
                ring[i % AHEAD] = operand(pv, qk, i + AHEAD, vslot, vhalf, kslot_q, khalf);
            else
                prefetch(i + AHEAD - NM);
            if constexpr (NEXT) {
#pragma unroll
                for (int r = i * CALLS / OVER; r < (i + 1) * CALLS / OVER; ++r)
                    if (r < CALLS) vector_work(r);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NEXT) sums_n = sums;
    };
    // A half with weights that are infinite or NaN.  In add_weights both columns of a pair would lose their sums, as 0 * inf and
    // 0 * NaN are NaN: a column whose own sum, of its two lanes, is not finite takes part in the product with weights of 0, and its
    // own sum is put in its place.  The other column's sum has the bits that it has beside finite weights.  Once the reference has
    // moved only a score of NaN or +inf comes to that, and the column's running sum is NaN from here on: its query becomes 0, so
    // that the halves to come do not end here again.
    auto keep_apart = [&](const u32x4 (&P)[2], f32x4 &sums) {
        float own = 0.f;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int w = 0; w < 4; ++w) own = sum2_bf16(P[q][w], own);
        float x, y;
        swap32(own, x, y);
        own = x + y;
        const bool lost = !(own <= 3.402823466e38f);   // (weights are not negative)
        sums = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 2; ++q) add_weights(u32x4{lost ? 0u : P[q][0], lost ? 0u : P[q][1], lost ? 0u : P[q][2], lost ? 0u : P[q][3]}, sums);
        own = lost ? own : 0.f;
        sums[0] += __shfl(own, lane & 15);
        sums[1] += __shfl(own, 16 + (lane & 15));
        m = lost ? 0.f : m;
        const uint32_t keep = lost ? 0u : ~0u;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qb[ks] &= keep;
    };
    // The reference that the weights of a half were computed with was too low for some column of the wave: move that of all its
    // columns to the maximum of the half and a margin, and compute the weights again.  With the margin scores may rise by 2^11 to
    // 2^16 before the next move.  The maximum itself keeps a weight that is a power of two, without a rounding error: moves by
    // powers of two, of weights that are only scaled, were faster yet (677 us for the last column below), but their errors on rising
    // scores 2 to 11 % larger.  All columns move together because every move costs the wave the same: columns that each move by
    // themselves took 715 / 634 us for the first two columns below.  So the rounding of an output can depend on the scores of the
    // other rows and heads of its wave, where those rise that far.
    // MI355X (us), 2 x 2048 rows on 4096 tokens, 64/8 heads; scores that rise by 2^72 over all keys / of deviation 4 / that rise by
    // 2^32 in every half / of deviation 1: maxima of every step and a rescale where one grew by 2^8, as the lean kernels do,
    // 585 / 613 / 581 / 598; no margin 558 / 592 / 741 / 560; as here 541 / 575 / 751 / 559.
    auto move_reference = [&](const f32x16 &Ss, u32x4 (&Pn)[2], f32x4 &sums_n) {
        float x, y;
        swap32(max16(Ss), x, y);
        const float m_new = max2(m, floor_m1e30(max2(x, y) * c_log2e) + kMargin);
        const float alpha = fast_exp2(m - m_new);
        m = m_new;
        weights16(Ss, Pn, sums_n);
        lsum_lo *= __shfl(alpha, lane & 15);
        lsum_hi *= __shfl(alpha, 16 + (lane & 15));
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[mb][r] *= alpha;
        if (too_large(sums_n)) keep_apart(Pn, sums_n);
    };

    const auto yes = std::true_type();
    const auto no = std::false_type();
    auto nothing = [](int) {};
    auto first_operands = [&](auto pv, auto qk, int vslot, int vhalf, int kslot_q, int khalf) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) ring[i] = operand(pv, qk, i, vslot, vhalf, kslot_q, khalf);
    };
    // The loads of a step, a wave's pieces of K beside the first MFMA of a region and those of V beside MFMA `later`: all of them at
    // once, at the start of a step, hold up the waves that issue them (860 cycles a step) and those of the unit's other workgroup.
    auto spread_issue = [&](int later, int i, int kslot_q, int k_id, int vslot, int v_id) {
        if (i == 0) issue(false, kslot_q, k_id);
        if (i == later) issue(true, vslot, v_id);
    };
    // the reference of the first half
    auto first_reference = [&](const f32x16 &S) {
        float x, y;
        swap32(max16(S), x, y);
        m = floor_m1e30(max2(x, y) * c_log2e);
    };

    if constexpr (PIPE && HV == 2) {
        // Two halves of 32 tokens per step.  P0, P1: weights of the halves of step st; S0, S1: their scores, and those of step st + 1
        // once the former have been used.  K runs one step ahead of V.
        f32x16 S0, S1;
        u32x4 P0[2], P1[2];
        f32x4 sums0, sums1;
        // Everybody's loads of K[st + 1] and V[st] have landed, and everybody is done with K[st] and V[st - 1].
        auto arrive = [&](int st) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __syncthreads();
            if (st * STEP + STEP > seq_len) scrub_v(st & 1, st * STEP);
        };
        auto roll_ids = [&](int st) {
            id1 = id2;
            id2 = next_id(st + 3);
        };
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("" : "+v"(idv), "+v"(idn));   // (arrived, and not to be waited for in the loop)
        __syncthreads();
        phase(2);
        first_operands(no, yes, 0, 0, st_lo & 1, 0);
        region(no, yes, no, P0, sums0, 0, 0, S0, P0, sums0, S0, st_lo & 1, 0, [&](int i) { ring[i] = operand(no, yes, i, 0, 0, st_lo & 1, 1); }, nothing);
        mask16(S0, st_lo * STEP);
        first_reference(S0);
        region(no, yes, yes, P0, sums0, 0, 0, S0, P0, sums0, S1, st_lo & 1, 1, nothing, nothing);
        if (too_large(sums0)) keep_apart(P0, sums0);
        // w_last: the last step that this wave has columns for; the loop runs to the one before
        const int w_last = w_used ? min(nstep - 1, w_pos_hi / T) : st_lo - 1;
        int st = st_lo;
        arrive(st);
        if (st < w_last) first_operands(yes, yes, st & 1, 0, (st + 1) & 1, 0);
        for (; st < w_last; ++st) {
            const int tok0 = st * STEP, cur = st & 1, nxt = (st + 1) & 1;
            if (tok0 + 63 > w_pos_lo) mask16(S1, tok0 + 32);
            // (the loads of K[st + 2], of any block if there is no such step, and V[st + 1])
            region(yes, yes, yes, P0, sums0, cur, 0, S1, P1, sums1, S0, nxt, 0, [&](int i) { ring[i] = operand(yes, yes, i, cur, 1, nxt, 1); },
                   [&](int i) { spread_issue(KS, i, cur, id2, nxt, id1); });
            if (too_large(sums1)) move_reference(S1, P1, sums1);
            roll_ids(st);
            if (tok0 + 95 > w_pos_lo) mask16(S0, tok0 + 64);
            // (the step's last operands are on their way when the next step's are waited for, whose first then follow them)
            region(yes, yes, yes, P1, sums1, cur, 1, S0, P0, sums0, S1, nxt, 1, [&](int i) { ring[i] = operand(yes, yes, i, nxt, 0, cur, 0); },
                   [&](int i) {
                       if (i == 2 * KS - AHEAD) arrive(st + 1);
                   });
            if (too_large(sums0)) move_reference(S0, P0, sums0);
        }
        if (st == w_last) {
            const int tok0 = st * STEP, cur = st & 1;
            if (st + 2 < nstep) issue(false, cur, id2);
            if (st + 1 < nstep) issue(true, (st + 1) & 1, id1);
            roll_ids(st);
            first_operands(yes, no, cur, 0, 0, 0);
            if (tok0 + 63 > w_pos_lo) mask16(S1, tok0 + 32);
            region(yes, no, yes, P0, sums0, cur, 0, S1, P1, sums1, S0, 0, 0, [&](int i) { ring[i] = operand(yes, no, i, cur, 1, 0, 0); }, nothing);
            if (too_large(sums1)) move_reference(S1, P1, sums1);
            region(yes, no, no, P1, sums1, cur, 1, S0, P0, sums0, S1, 0, 0, nothing, nothing);
            ++st;
            if (st < nstep) arrive(st);
        }
        for (; st < nstep; ++st) {   // steps that other waves have columns for: this one stages only
            if (st + 2 < nstep) issue(false, st & 1, id2);
            if (st + 1 < nstep) {
                issue(true, (st + 1) & 1, id1);
                roll_ids(st);
                arrive(st + 1);
            }
        }
    } else if constexpr (PIPE) {
        // One half per step.  Step st multiplies the weights of step st - 1, turns the scores of step st into weights and computes
        // those of step st + 1: V runs two steps behind K.
        static_assert(HV == 1, "a half per step");
        f32x16 SA, SB;
        u32x4 PA[2], PB[2];
        f32x4 sumsA, sumsB;
        // Everybody's loads of K[st + 1] and V[st - 1] have landed, and everybody is done with K[st] and V[st - 2].
        auto arrive = [&](int st) {
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __syncthreads();
            if (st > st_lo && st * STEP > seq_len) scrub_v((st - 1) & 1, (st - 1) * STEP + kg * T);
        };
        auto roll_ids = [&](int st) {
            id0 = id1;
            id1 = id2;
            id2 = next_id(st + 3);
        };
        auto load_step = [&](int st) {   // K[st + 2] and V[st]
            if (st + 2 < nstep) issue(false, st & 1, id2);
            if (st > st_lo && st < nstep) issue(true, st & 1, id0);
            roll_ids(st);
        };
        auto mask_step = [&](f32x16 &S, int st) {
            if (st * STEP + kg * T + T - 1 > w_pos_lo) mask16(S, st * STEP + kg * T);
        };
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        asm volatile("" : "+v"(idv), "+v"(idn));
        __syncthreads();
        phase(2);
        first_operands(no, yes, 0, 0, st_lo & 1, 0);
        region(no, yes, no, PA, sumsA, 0, 0, SA, PA, sumsA, SA, st_lo & 1, 0, nothing, nothing);
        // w_last: the last step that this wave has columns for
        const int w_last = w_pos_hi >= kg * T ? min(nstep - 1, (w_pos_hi - kg * T) / STEP) : st_lo - 1;
        int st = st_lo;
        arrive(st);
        if (st <= w_last) {
            mask_step(SA, st);
            first_reference(SA);
            if (st < w_last) {
                first_operands(no, yes, 0, 0, (st + 1) & 1, 0);
                load_step(st);
                region(no, yes, yes, PA, sumsA, 0, 0, SA, PA, sumsA, SB, (st + 1) & 1, 0, nothing, nothing);
                if (too_large(sumsA)) keep_apart(PA, sumsA);
                ++st;
                arrive(st);
                if (st < w_last) first_operands(yes, yes, (st - 1) & 1, 0, (st + 1) & 1, 0);
                // one step: scores Ss and weights Pu of the step before, which leave scores Sq and weights Pn; the loads are K[st + 2] (of
                // any block if there is no such step) and V[st]
                auto full = [&](f32x16 &Ss, f32x16 &Sq, u32x4 (&Pu)[2], f32x4 &sums_u, u32x4 (&Pn)[2], f32x4 &sums_n) {
                    const int cur = st & 1, nxt = (st + 1) & 1;
                    mask_step(Ss, st);
                    // (the loads have one step: they are waited for at its end, not where the last operands are on their way, 0.95 of the
                    // time on long contexts)
                    region(yes, yes, yes, Pu, sums_u, nxt, 0, Ss, Pn, sums_n, Sq, nxt, 0, nothing, [&](int i) { spread_issue(KS / 2, i, cur, id2, cur, id0); });
                    if (too_large(sums_n)) move_reference(Ss, Pn, sums_n);
                    roll_ids(st);
                    ++st;
                    arrive(st);
                    if (st < w_last) first_operands(yes, yes, cur, 0, cur, 0);
                };
                while (st < w_last) {
                    full(SB, SA, PA, sumsA, PB, sumsB);
                    if (st >= w_last) {
                        SB = SA;
                        PA[0] = PB[0];
                        PA[1] = PB[1];
                        sumsA = sumsB;
                        break;
                    }
                    full(SA, SB, PB, sumsB, PA, sumsA);
                }
                first_operands(yes, no, (st - 1) & 1, 0, 0, 0);
                load_step(st);
                mask_step(SB, st);
                region(yes, no, yes, PA, sumsA, (st - 1) & 1, 0, SB, PB, sumsB, SA, 0, 0, nothing, nothing);
            } else {
                load_step(st);
                SB = SA;
                weights16(SB, PB, sumsB);
            }
            if (too_large(sumsB)) move_reference(SB, PB, sumsB);
            ++st;
            arrive(st);
            first_operands(yes, no, (st - 1) & 1, 0, 0, 0);
            load_step(st);
            region(yes, no, no, PB, sumsB, (st - 1) & 1, 0, SA, PB, sumsB, SB, 0, 0, nothing, nothing);
        } else {
            load_step(st);
        }
        for (; st < nstep; ++st) {   // steps that other waves have columns for: this one stages only
            arrive(st + 1);
            load_step(st + 1);
        }
    } else {
        // No pipeline across steps (few registers, see prefill_kernel_lean): scores, weights and product of a step one after the other,
        // the overlap of matrix and vector work comes from the two waves of a SIMD.
        float lsum = 0.f;
        m = -INFINITY;
        // scores of one step: S[hh] register r is token st*64 + 32hh + 8h + 16(r/8) + r%8
        auto qk = [&](f32x16 (&S)[HV], int slot) {
#pragma unroll
            for (int hh = 0; hh < HV; ++hh)
#pragma unroll
                for (int r = 0; r < 16; ++r) S[hh][r] = 0.f;
            // the two token halves alternate, so that consecutive MFMAs never wait for each other's result
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int hh = 0; hh < HV; ++hh) {
                    const u32x4 kop = ldsK[slot][(2 * hh + ku) * CH + (2 * ks + h) * 16 + kslot];
                    S[hh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop),
                                                                __builtin_bit_cast(bf16x8, qb[ks]), S[hh], 0, 0, 0);
                }
        };
        // causal mask of a step that touches the diagonal
        auto mask = [&](f32x16 (&S)[HV], int tok0) {
            const int room = pos - (tok0 + 8 * h);           // visible iff 32hh + 16(r/8) + r%8 <= room
#pragma unroll
            for (int hh = 0; hh < HV; ++hh)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    S[hh][r] = (32 * hh + 16 * (r / 8) + (r % 8) <= room) ? S[hh][r] : -INFINITY;
        };
        // online-softmax update with the raw scores of one step; P[2hh+u] holds the packed weights of
        // tokens 32hh + 16u + 8h + 0..7.  The softmax scale rides in the fma that feeds exp2 (scale > 0,
        // so the maximum can be taken before scaling).
        // The update comes in two halves so that the PV products of the first 32 tokens can run beside the
        // exponentials of the last 32: weights(S, P, q4, ...) turns the scores of tokens 16*q4 + 8h + 0..7 into P[q4].
        auto weights = [&](const f32x16 (&S)[HV], u32x4 (&P)[2 * HV], int q4, float m_ref, float &psum) {
            float e[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) e[r] = fast_exp2(__builtin_fmaf(S[q4 >> 1][8 * (q4 & 1) + r], c_log2e, -m_ref));
            P[q4] = u32x4{pack2_bf16(e[0], e[1]), pack2_bf16(e[2], e[3]), pack2_bf16(e[4], e[5]), pack2_bf16(e[6], e[7])};
            // the denominator sums the same rounded weights that enter the PV product
#pragma unroll
            for (int w = 0; w < 4; ++w) psum = sum2_bf16(P[q4][w], psum);
        };
        auto softmax_first = [&](const f32x16 (&S)[HV], u32x4 (&P)[2 * HV], float &alpha, bool &grow, float &psum) {
            float mloc;
            if constexpr (HV == 2)
                mloc = max32(S[0], S[1]);
            else
                mloc = max16(S[0]);
            {
                float x, y;
                swap32(mloc, x, y);
                mloc = max2(x, y) * c_log2e;
            }
            // (floored: a part of a split tile may start with steps that a column does not see at all; its maximum
            // then stays at the floor, its weights and sum at 0, instead of running into inf - inf)
            // The reference point m only has to stay within 2^8 of the true running maximum (weights up to 256 are
            // exact enough in bf16 and harmless in the fp32 sums; the final division cancels the reference), so it
            // moves, and the accumulators are rescaled, only when a step's maximum exceeds it by more than 8.
            const float m_cand = floor_m1e30(mloc);
            grow = m_cand > m + 8.0f;
            const float m_new = grow ? m_cand : m;
            alpha = fast_exp2(m - m_new);
            m = m_new;
            psum = 0.f;
#pragma unroll
            for (int q = 0; q < HV; ++q) weights(S, P, q, m, psum);
        };
        auto softmax_second = [&](const f32x16 (&S)[HV], u32x4 (&P)[2 * HV], float alpha, float psum) {
#pragma unroll
            for (int q = HV; q < 2 * HV; ++q) weights(S, P, q, m, psum);
            lsum = lsum * alpha + psum;
        };
        for (int st = st_lo; st < nstep; ++st) {
            // the loads of K[st] and V[st] have landed (everybody's, after the barrier); nobody reads the tiles of
            // step st-1 any more, so the loads of step st+1 may overwrite them
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (st + 1 < nstep) {
                issue_apart(false, (st + 1) & 1, id1, id1b);
                issue_apart(true, (st + 1) & 1, id1, id1b);
            }
            const int tok0 = st * STEP + kg * T;
            if (st * STEP + STEP > seq_len) scrub_v(st & 1, tok0);
            id1 = ctable[min(wave_block(st + 2), nblk - 1)];
            id1b = ctable[min(wave_block(st + 2) + 2, nblk - 1)];
            if (tok0 > w_pos_hi) continue;   // wave-uniform: no column of this wave sees keys of the step
            f32x16 S[HV];
            qk(S, st & 1);
            if (tok0 + T - 1 > w_pos_lo) mask(S, tok0);
            u32x4 P[2 * HV];
            float alpha, psum;
            bool grow;
            softmax_first(S, P, alpha, grow, psum);
            if (__any(grow)) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) O[mb][r] *= alpha;
            }
            softmax_second(S, P, alpha, psum);
            const u32x4 *vp = &ldsV[st & 1][h * HD + col];
#pragma unroll
            for (int i = 0; i < 2 * HV * MB; ++i) {
                const u32x4 vop = vp[(i / MB) * CH + 32 * (i % MB)];
                O[i % MB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vop),
                                                                __builtin_bit_cast(bf16x8, P[i / MB]), O[i % MB], 0, 0, 0);
            }
        }
        float x, y;
        swap32(lsum, x, y);
        lsum_lo = lsum_hi = x + y;
    }
    float ltot = (lane & 16) ? lsum_hi : lsum_lo;
    phase(3);
    if (phases && tid == 0) *phases = phase_bits;
    // Piece q of a wave's output (0 .. 4*MB-1) is, in lane (col, h), column 32*wave + col, dims 8q + 4h + 0..3: registers
    // 4*(q % 4) .. + 3 of O[q / 4].  From here on a thread holds ITEMS pieces of its column, q0 .. q0 + ITEMS - 1.
    const int q0 = KG == 1 ? 0 : kg * ITEMS;
    f32x4 acc[ITEMS];
    if constexpr (KG == 1) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) acc[i] = f32x4{O[i / 4][4 * (i % 4)], O[i / 4][4 * (i % 4) + 1], O[i / 4][4 * (i % 4) + 2], O[i / 4][4 * (i % 4) + 3]};
    } else {
        // The key groups' results meet in the stage memory, which they fill exactly: every wave writes all its pieces, and
        // the KG waves of a column group each fold the pieces of one KG-th of the dims, in the order of the groups.
        __shared__ f32x2 group_ml[NW][32];
        static_assert(NW * 4 * MB * 64 == 4 * KG * STAGE, "the results fill the stage memory");
        f32x4 (*const all)[4 * MB][64] = reinterpret_cast<f32x4 (*)[4 * MB][64]>(stage_lds<HD, KG>());
        __syncthreads();   // nobody reads K or V tiles any more
#pragma unroll
        for (int q = 0; q < 4 * MB; ++q)
            all[wave_id][q][lane] = f32x4{O[q / 4][4 * (q % 4)], O[q / 4][4 * (q % 4) + 1], O[q / 4][4 * (q % 4) + 2], O[q / 4][4 * (q % 4) + 3]};
        if (h == 0) group_ml[wave_id][col] = f32x2{m, ltot};
        __syncthreads();
        f32x2 ml[KG];
        float M = -1e30f;   // (finite: no group may have seen a key of this column, which then weighs nothing)
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            ml[k] = group_ml[k * NC + wave][col];
            M = fmaxf(M, ml[k][0]);
        }
        ltot = 0.f;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < KG; ++k) {
            const float w = fast_exp2(ml[k][0] - M);
            ltot += ml[k][1] * w;
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) {
                const f32x4 o = all[k * NC + wave][q0 + i][lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][r] += o[r] * w;
            }
        }
        m = M;
    }
    // This wave's pieces first .. of its columns, divided by the sums, to the output: through LDS, so that a store instruction
    // writes whole rows (pieces of one wave are side by side) and not 16 bytes of each of 32.  The stage memory is free.  A piece
    // is 16 bytes of the output; those of a column lie in LDS with their index permuted by the column, which spreads a wave's
    // writes over the banks.
    // Why that is faster than stores of 8 bytes per lane, 16 to a row of 256 bytes, the counters do not say: either way the bytes that
    // reach memory are those of the output.  Past the caches (`nt`) it is faster again, where the output is read next as well (attention
    // and a projection of a captured layer, 8 x 512 rows beside 128 decodes 326 -> 313; level or up to 2 % better elsewhere, a plain
    // copy of the output behind 2000 rows of prompts 30.7 -> 31.1).
    // MI355X (us), 8 bytes per lane -> rows -> rows, nt: 8 x 512 rows beside 128 decodes 262.0 -> 257.6 -> 242.6, 2 x 2048 rows beside
    // 32 long decodes 1647 -> 1631 -> 1559, 8 x 512 rows alone 81.5 -> 79.4 -> 78.4, six prompts of 295 rows 16.2 -> 14.4 -> 13.0;
    // without any output stores the first two take 226 and 1533.  (Key groups, whose waves have a quarter of each row: 2 x 133 rows on
    // 1231 tokens 17.9 -> 17.3; 24 decodes beside 237 rows lose 1.6 % with `nt` on such quarters.)
    auto put = [&](const auto &a, int first) {
        constexpr int N = std::extent_v<std::remove_reference_t<decltype(a)>>, PASS = 64 / N;   // rows of a store instruction
        static_assert(N >= 2 && N <= 16 && (N & (N - 1)) == 0, "a permutation of N pieces");
        auto place = [&](int column, int piece) -> int { return column * N + (piece ^ ((column / (16 / N)) & (N - 1))); };
        u32x4 *const rows_lds = stage_lds<HD, KG>() + wave_id * 32 * N;
        const float inv = 1.0f / ltot;
#pragma unroll
        for (int i = 0; i < N; ++i)
            reinterpret_cast<u32x2 *>(rows_lds + place(col, i))[h] =
                u32x2{pack2_bf16(a[i][0] * inv, a[i][1] * inv), pack2_bf16(a[i][2] * inv, a[i][3] * inv)};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int n = 0; n < 32 / PASS; ++n) {
            const int r = n * PASS + lane / N, piece = lane % N;
            const u32x4 w = rows_lds[place(r, piece)];
            const int cc = wave * 32 + r, cc_row = (int)((uint32_t)cc * p.g_magic >> 15), cc_head = cc - cc_row * g;
            if (cc_row < rows) {
                u32x4 *const dst = reinterpret_cast<u32x4 *>(p.out + ((int64_t)(q_row0 + cc_row) * p.Hq + kvh * g + cc_head) * HD + 8 * (q0 + first + piece));
                if constexpr (KG == 1)
                    __builtin_nontemporal_store(w, dst);
                else   // (a quarter of a row: 64 bytes of a line)
                    *dst = w;
            }
        }
        __builtin_amdgcn_wave_barrier();   // (before the next pieces)
    };
    if (nparts > 1) {
        // (one counter per (tile, kv head): the slot of its part 0 with the list, the unit's index without)
        const int counter_idx = p.pf_table ? slot0 : slot0 / split;
        // ---- partial result of this part, arrival count, merge by the part that arrives last (same
        // device-scope accesses as the decode kernel).  Layout of a part: [wave of columns][piece][lane][4 floats], so that
        // every store and load instruction of a wave covers 1 KiB of contiguous memory.  Waves without columns have nothing
        // to store or merge (a chunk of 5 rows x 4 heads: one wave's 16 KiB instead of 64).
        auto part_ptr = [&](int64_t j) -> float * {
            return p.pf_acc + (((int64_t)(slot0 + (int)j * slot_step) * NC + wave) * 4 * MB + q0) * 256 + lane * 4;
        };
        auto ml_ptr = [&](int64_t j) -> float * { return p.pf_ml + ((int64_t)(slot0 + (int)j * slot_step) * COLS + c) * 2; };
        if (w_used) {
            float *const pp = part_ptr(part);
#pragma unroll
            for (int i = 0; i < ITEMS; ++i) store_dev4(pp + i * 256, acc[i]);
            if (h == 0 && kg == 0) store_dev2(ml_ptr(part), m, ltot);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partial has reached memory ...
        __syncthreads();                                    // ... and so have the other waves'
        // Pieces first .. first + N - 1 (of this thread's) of all parts, in part order: the result does not depend on who is
        // last or who merges.  16 loads of a lane on their way at a time: 16 / N parts.
        auto merge = [&](auto &a, int first) {
            constexpr int N = std::extent_v<std::remove_reference_t<decltype(a)>>, PB = 16 / N;
            float M = -INFINITY;
            ltot = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int j0 = 0; j0 < nparts; j0 += PB) {
                f32x2 ml[PB];
                f32x4 t[16];
#pragma unroll
                for (int b = 0; b < PB; ++b) ml[b] = load_dev2(ml_ptr(min(j0 + b, nparts - 1)));
                auto pp = [&](int b) -> const float * { return part_ptr(min(j0 + b, nparts - 1)) + first * 256; };
                if constexpr (PB == 1)
                    load_dev_part<4>(t, pp(0), pp(0) + 1024, pp(0) + 2048, pp(0) + 3072);
                else if constexpr (PB == 2)
                    load_dev_part<4>(t, pp(0), pp(0) + 1024, pp(1), pp(1) + 1024);
                else if constexpr (PB == 4)
                    load_dev_part<4>(t, pp(0), pp(1), pp(2), pp(3));
                else
                    load_dev_part<2>(t, pp(0), pp(1), pp(2), pp(3), pp(4), pp(5), pp(6), pp(7));
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    if (j0 + b < nparts) {
                        const float M_new = fmaxf(M, ml[b][0]);
                        const float w_old = fast_exp2(M - M_new), w_new = fast_exp2(ml[b][0] - M_new);
                        M = M_new;
                        // (the fused multiply-adds are spelled out: every N gives the same bits)
                        ltot = __builtin_fmaf(ltot, w_old, ml[b][1] * w_new);
#pragma unroll
                        for (int i = 0; i < N; ++i)
#pragma unroll
                            for (int r = 0; r < 4; ++r) a[i][r] = __builtin_fmaf(a[i][r], w_old, t[b * N + i][r] * w_new);
                    }
                }
            }
        };
        __shared__ int arrived;
        int32_t *const counter = p.pf_counters + counter_idx;
        if constexpr (KG == 1 && PIPE) {
            if (p.pf_share && nparts >= kSharedMergeParts) {
                // The merge of a tile of many parts is shared: the parts end within a few microseconds of each other, and one
                // unit reads 64 KB of partial results in 1.2 us, a part after the other (six parts 8 .. 11 us at the end of
                // the launch, eleven 15).  So a part that ends early waits, for a bounded time, until the last one has arrived;
                // the dims fall into MergeWord::kSlices slices, the last part takes the first and whoever is there draws the others.
                // Only where all workgroups of the launch find a place at once, so that nobody waits for the place of one that
                // waits -- unless another stream's work holds units: hence the bound.
                // MI355X (us, one merging part -> shared): 11 parts, 2 x 74 rows on 13,000 tokens, 28/4 heads 45.5 -> 42.0; drawn
                // batches of 5 .. 16 parts 13.0 -> 11.8, 39.2 -> 36.7, 86.0 -> 79.6; six parts of 80 tiles, whose 32 MB of partial
                // results are a matter of HBM as well, 87.8 -> 86.9.  Eight slices lose half of that; looks at the counter every
                // 1.2 us instead of 2 slow down the parts that still work (67 -> 70 us for the steps of those six parts).
                constexpr int PI = ITEMS / MergeWord::kSlices;
                static_assert(kMaxPrefillSplit + MergeWord::kSlices < 256, "a byte each");
                auto event = [&](int what) -> int {   // the word that it found
                    const int w = __hip_atomic_fetch_add(counter, what, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (MergeWord::last_event(w, nparts)) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return w;
                };
                auto draw = [&]() -> int { return MergeWord::slice(event(MergeWord::kDraw)); };
                if (tid == 0) {
                    const int w = __hip_atomic_fetch_add(counter, MergeWord::kArrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    int mine = 0;
                    if (!MergeWord::arrived_last(w, nparts)) {
                        bool all = false;
                        for (int i = 1; i < p.pf_share && !all; ++i) {   // (a load and a pause: 2 us or so)
                            __builtin_amdgcn_s_sleep(40);
                            all = MergeWord::arrivals(__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == nparts;
                        }
                        if (all) {
                            mine = draw();
                        } else {
                            (void)event(MergeWord::kLeave);
                            mine = -1;
                        }
                    }
                    arrived = mine;
                }
                for (;;) {
                    __syncthreads();
                    const int slice = __builtin_amdgcn_readfirstlane(arrived);
                    if (slice < 0) return;
                    if (w_used) {
                        f32x4 a[PI];
                        merge(a, slice * PI);
                        put(a, slice * PI);
                    }
                    __syncthreads();   // everybody has read `arrived`
                    if (tid == 0) arrived = draw();
                }
            }
        }
        if (tid == 0) arrived = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (arrived != nparts - 1) return;
        if (tid == 0)   // ready for the next call
            __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!w_used) return;
        merge(acc, 0);
    } else {
        __syncthreads();   // nobody reads the stage memory any more
    }
    put(acc, 0);
}

// The tile list's word of this workgroup's row (see AttnParams::list_row): its address needs no other argument.
OOCO_DEV int row_word(const KernArgs &a) { return a.cum[kInlineSeqs - min((int)blockIdx.y, kInlineSeqs)]; }
// (What a prefill workgroup needs of the arguments before its first tile, asked for together: see decode_kernel_body.)
OOCO_DEV void prefill_args(const AttnParams &p)
{
    asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.block_tables), "s"(p.seq_lens), "s"(p.query_start_loc),
                 "s"(p.ctx_lens), "s"(p.trace), "s"(p.Hq), "s"(p.Hkv), "s"(p.g), "s"(p.max_blocks_per_seq), "s"(p.num_seqs),
                 "s"(p.total_q), "s"(p.scale_log2e), "s"((int)p.pf_table), "s"((int)p.g_magic), "s"((int)p.list_by_seq));
}

template <int HD, int NW, int KG>
OOCO_DEV void prefill_kernel_body(const KernArgs &a)
{
    const AttnParams &p = a.p;
    int tile_word = row_word(a);
    prefill_args(p);
    const int vb = (int)(blockIdx.y * (unsigned)p.Hkv + blockIdx.x);
    // option "trace" on a batch without decode work: per workgroup (start, XCD * 256 + compute unit id, times of
    // four phases since the start, end)
    uint64_t *const trace = (p.trace && p.static_runs == 0) ? p.trace + (int64_t)vb * 4 : nullptr;
    const uint64_t t_start = trace ? wall_clock64() : 0;
    if (trace && threadIdx.x == 0) {
        trace[0] = t_start;
        trace[1] = (__builtin_amdgcn_s_getreg((31 << 11) | 20) & 7u) * 256u + ((__builtin_amdgcn_s_getreg((31 << 11) | 4) >> 8) & 255u);
        trace[2] = 0;   // (a workgroup that leaves before its first step stores no phases)
    }
    if (!p.list_by_seq && p.pf_table) tile_word = plan_entry(a, 2 * p.num_pf + 1 + (int)blockIdx.y);
    prefill_unit<HD, NW, true, KG>(p, [&](int idx) -> int { return plan_entry(a, idx); }, vb, (int)blockIdx.y, (int)blockIdx.x, tile_word,
                                   trace ? trace + 2 : nullptr, t_start);
    if (trace) {
        __syncthreads();
        if (threadIdx.x == 0) trace[3] = wall_clock64();
    }
}
template <int HD, int NW>
__global__ __launch_bounds__(NW * 64, HD == 64 ? 3 : 8 / NW) void prefill_kernel(const KernArgs a)
{
    prefill_kernel_body<HD, NW, 1>(a);
}
template <int HD>
__global__ __launch_bounds__(512, 1) void prefill_kernel_groups(const KernArgs a)
{
    prefill_kernel_body<HD, 8, kKeyGroups>(a);
}

// Eight waves, 256 query columns, no software pipeline, at most 176 registers per wave: the prefill kernel of
// batches that also hold decode work (see decode_kernel_lean).
template <int HD>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_num_vgpr(168))) void prefill_kernel_lean(const KernArgs a)
{
    const AttnParams &p = a.p;
    int tile_word = row_word(a);
    prefill_args(p);
    if (!p.list_by_seq && p.pf_table) tile_word = plan_entry(a, 2 * p.num_pf + 1 + (int)blockIdx.y);
    prefill_unit<HD, 8, false, 1>(p, [&](int idx) -> int { return plan_entry(a, idx); }, (int)(blockIdx.y * (unsigned)p.Hkv + blockIdx.x),
                                  (int)blockIdx.y, (int)blockIdx.x, tile_word);
}

// ------------------------------------------------------------------------------------------
// Both kinds of work of a step in ONE launch: the first p.dec_wgs workgroups are decode waves (up to four per workgroup, each
// one (run, kv head) item of the decode line, exactly as in the decode kernel), the others prefill workgroups (exactly
// as in the prefill kernel).  Every unit holds both kinds side by side as with two kernels on two streams, without the
// fork and join events of the second stream, and a short batch does not wait for one kernel to drain before the other
// starts.  Decode workgroups come first in dispatch order, so that each unit gets its share of the HBM stream before
// prefill workgroups fill it up.  Against the two kernels on two streams, MI355X: a call on an idle GPU 297 -> 283 us (8 x 512
// rows + 128 decodes) and 1653 -> 1635 (2 x 2048 + 32 long decodes); in a loop of calls level, 266 / 268 and 1625 / 1630, but
// 340 and 2170 on a context whose side stream shares a hardware queue with the caller's stream (one or two of eight contexts
// made in a row), where the kernels run in sequence.  2 x 120 rows + 24 short decodes, in sequence before: 37.5 -> 29.
// DEC = decode's KV blocks: of a step (single waves), or in flight (cooperative workgroups, see decode_coop_run).
template <int HD, int DEC, int MBATCH, int NW, bool PIPE, bool COOP, int KG = 1>
OOCO_DEV void step_body(const KernArgs &a)
{
    const AttnParams &p = a.p;
    int tile_word = row_word(a);
    prefill_args(p);
    const int wg = p.rows2d ? (int)(blockIdx.y * (unsigned)p.Hkv + blockIdx.x) : (int)blockIdx.x;
    if (COOP && wg < p.dec_wgs) {   // cooperative decode workgroups
        static_assert(!COOP || kCoopFloats<HD, NW> * sizeof(float) <= 4 * KG * kPfGroupBlocks<KG> * HD * 2 * sizeof(u32x4), "fits the stage memory");
        const int run = p.rows2d ? (int)blockIdx.y : wg / p.Hkv, slot = wg - run * p.Hkv;
        uint64_t *const trace = p.trace ? p.trace + (int64_t)wg * 4 : nullptr;
        if (trace && threadIdx.x == 0) trace[0] = wall_clock64();
        decode_coop_run<HD, COOP ? DEC : 256 / HD, NW>(p, [&](int idx) -> int { return a.cum[idx]; }, a.cum[1 + (threadIdx.x & 63)], run,
                                     p.rotate_heads ? (slot + run) % p.Hkv : slot,
                                     reinterpret_cast<float *>(stage_lds<HD, KG>()), trace);
        if (trace) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (threadIdx.x == 0) trace[3] = wall_clock64();
        }
    } else if (!COOP && wg < p.dec_wgs) {
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        // (the waves of a workgroup take items far apart: side by side they hold the kv heads of one run, finish together and
        // merge one long sequence's parts on one unit, which reads no faster for three waves than for one -- a sequence of
        // 73,000 tokens in 80 parts, 64/8 heads: 52 us from the last step to the end, and 26 apart)
        const int item = p.dec_near ? wg * p.dec_wpw + wave : wave * p.dec_wgs + wg;
        if (wave >= p.dec_wpw || item >= p.static_runs * p.Hkv) return;
        asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.block_tables), "s"(p.seq_lens),
                     "s"(p.query_start_loc), "s"(p.Hq), "s"(p.Hkv), "s"(p.g), "s"(p.max_blocks_per_seq), "s"(p.num_seqs),
                     "s"(p.total_q), "s"(p.dec_blocks), "s"(p.static_blocks), "s"(p.static_runs), "s"(p.piece_pad),
                     "s"((int)p.rotate_heads), "s"(p.scale_log2e), "s"(p.trace));
        const int lane = (int)threadIdx.x & 63;
        const int run = item / p.Hkv, slot = item - run * p.Hkv;
        const int kvh = p.rotate_heads ? (slot + run) % p.Hkv : slot;
        uint64_t *const trace = p.trace ? p.trace + (int64_t)item * 4 : nullptr;
        if (trace && lane == 0) trace[0] = wall_clock64();
        bool first_piece = true;
        decode_run<HD, DEC, MBATCH>(p, [&](int idx) -> int { return a.cum[idx]; }, a.cum[1 + lane], EqualRuns{p.static_blocks, p.static_runs},
                                    run, kvh, lane, trace, first_piece, []() {});
        if (trace) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) trace[3] = wall_clock64();
        }
    } else {
        const int n_cum = p.num_seqs + 1;   // the prefill array follows the decode array
        const int vb = wg - p.dec_wgs;
        int entry = (int)blockIdx.y - p.list_row, kvh = (int)blockIdx.x;
        if (!p.rows2d && p.pf_table) {
            entry = vb / p.Hkv;
            kvh = vb - entry * p.Hkv;
            tile_word = a.cum[kInlineSeqs - p.list_row - entry];
        }
        prefill_unit<HD, NW, PIPE, KG>(p, [&](int idx) -> int { return a.cum[n_cum + idx]; }, vb, entry, kvh, tile_word);
    }
}

template <int HD, int DEC, bool COOP>
__global__ __launch_bounds__(kPfThreads, HD == 64 ? 3 : 2) void step_kernel(const KernArgs a)
{
    step_body<HD, DEC, 3, 4, true, COOP>(a);
}

// The same with prefill workgroups of key groups and decode workgroups of eight waves, which have a compute unit each: small
// batches whose workgroups all find one.
template <int HD, int DEC>
__global__ __launch_bounds__(512, 1) void step_kernel_groups(const KernArgs a)
{
    step_body<HD, DEC, 3, 8, true, true, kKeyGroups>(a);
}

// The register-lean pair in one launch: prefill workgroups of eight waves; of a decode workgroup's eight waves the
// first four decode, one per SIMD, and the others leave at once, which frees their registers for the two prefill waves
// that the SIMD holds beside it (3 x 168 <= 512).
template <int HD>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_num_vgpr(168))) void step_kernel_lean(const KernArgs a)
{
    step_body<HD, 1, 1, 8, false, false>(a);
}

// ------------------------------------------------------------------------------------------
// Mixed batches in ONE launch: a persistent grid of two 256-thread workgroups per compute unit in which a compute
// unit runs EITHER decode waves (eight per unit, each streaming runs of the decode line exactly as the decode
// kernel's waves do) OR prefill workgroups (two per unit, each working through (tile, kv head) units exactly as
// the prefill kernel's workgroups do).  Side by side on one unit the two kinds get into each other's way -- the
// decode waves lose their issue slots and the matrix pipe to prefill waves that keep both busy, the prefill
// workgroups lose half their register file -- and both kernels stretch; apart, the decode units keep HBM busy
// while the prefill units keep the matrix cores busy.
//   * Which unit does what: the first workgroup to arrive on a compute unit (identified by the hardware's XCD,
//     shader-engine and CU ids) claims it and draws the unit's rank within its XCD from a counter; the other
//     workgroup of the unit reads that rank.  Ranks below p.dec_cus decode, the others prefill, so every XCD (and
//     its L2) gets the same mix.
//   * Work is pulled from counters: decode waves draw (run, kv head) items, prefill workgroups draw units from
//     the list of their own XCD first (unit index = XCD mod 8, so the tiles that share keys meet in one L2, as
//     in the stand-alone kernel) and from the other XCDs' lists after that.
//   * A workgroup whose own kind of work has run out takes up the other kind once, then leaves: the split of the
//     units only has to be roughly right.
// Nothing waits for another workgroup except the bounded look at a claim in progress, so the grid drains whatever
// the placement.  The last workgroup to leave resets the claims and counters for the next launch (or replay).
// State (int32, zero between launches), at p.queue - kMixedStateInts + 1:
//   [0, 2048) claims: 0 free, 1 being claimed, rank + 2;  [2048, 2056) arrivals per XCD;
//   [2056, 2064) prefill units drawn per XCD;  [2064] decode items drawn;  [2065] workgroups that have left
constexpr int kMixedClaims = 2048;
constexpr int kMixedShareCus = 99;
template <int HD>
__global__ __launch_bounds__(kPfThreads, 2) void mixed_kernel(const KernArgs a)
{
    const AttnParams &p = a.p;
    __shared__ int sh_role, sh_item;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    int32_t *const state = reinterpret_cast<int32_t *>(p.queue) - (kMixedStateInts - 1);
    int32_t *const claims = state, *const xcd_arrivals = state + kMixedClaims, *const pf_drawn = state + kMixedClaims + 8;
    int32_t *const dec_drawn = state + kMixedClaims + 16, *const left = state + kMixedClaims + 17;
    const int n_cum = p.num_seqs + 1;   // the prefill array follows the decode array
    auto dcum_at = [&](int idx) -> int { return p.cum_dev ? cum_entry<true>(a, idx) : cum_entry<false>(a, idx); };
    const int dcum_head = p.cum_dev ? cum_head<true>(a, lane) : cum_head<false>(a, lane);
    auto pf_at = [&](int idx) -> int { return plan_entry(a, n_cum + idx); };
    const unsigned xcc = __builtin_amdgcn_s_getreg((31 << 11) | 20) & 7u;              // XCC_ID
    if (tid == 0) {
        const unsigned hw = __builtin_amdgcn_s_getreg((31 << 11) | 4);                 // HW_ID: CU, SH, SE ids in bits 8..15
        int32_t *const claim = claims + (xcc * 256u + ((hw >> 8) & 255u));
        int expected = 0, rank;
        const bool won = __hip_atomic_compare_exchange_strong(claim, &expected, 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT);
        if (won) {
            rank = __hip_atomic_fetch_add(xcd_arrivals + xcc, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(claim, rank + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            // the claimant runs on this very compute unit and needs two more memory operations: a bounded look
            int v = expected;
            for (int spin = 0; v < 2 && spin < (1 << 16); ++spin) {
                __builtin_amdgcn_s_sleep(8);
                v = __hip_atomic_load(claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            rank = v >= 2 ? v - 2 : 0;   // (never seen: decode)
        }
        // p.dec_cus == kMixedShareCus: every unit runs both kinds side by side (its first workgroup decodes, its
        // second prefills) -- the arrangement of the two separate kernels, inside one launch, kept for measurements
        sh_role = p.dec_cus == kMixedShareCus ? (won ? 0 : 1) : (rank < p.dec_cus ? 0 : 1);
    }
    __syncthreads();
    int role = sh_role;   // 0 = decode, 1 = prefill
    // option "trace": per workgroup (start, end of its first kind of work, end of its second kind, first role +
    // 256 * items of wave 0 in the first kind + 2^32 * items in the second) on the 100 MHz clock
    uint64_t *const trace = p.trace ? p.trace + (int64_t)blockIdx.x * 4 : nullptr;
    uint64_t n_first = 0, n_second = 0;   // (two scalars: an array indexed by the pass would live in scratch memory)
    if (trace && tid == 0) {
        trace[0] = wall_clock64();
        trace[3] = (uint64_t)role;
    }
    const int n_dec_items = p.static_runs * p.Hkv;
    const int n_vb = p.pf_table ? p.pf_table * p.Hkv : p.n_tiles * p.Hkv * p.pf_split;
    const EqualRuns L = {p.static_blocks, p.static_runs};
    for (int pass = 0; pass < 2; ++pass, role ^= 1) {
        if (role == 0) {
            bool first_piece = false;
            for (;;) {
                int item = 0;
                if (lane == 0) item = __hip_atomic_fetch_add(dec_drawn, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                item = __builtin_amdgcn_readfirstlane(item);
                if (item >= n_dec_items) break;
                const int run = item / p.Hkv;
                const int kvh = (item - run * p.Hkv + run) % p.Hkv;   // kv heads rotate over the runs
                decode_run<HD, (HD == 64 ? 2 : 1), 3>(p, dcum_at, dcum_head, L, run, kvh, lane, nullptr, first_piece, []() {});
                if (pass == 0) ++n_first; else ++n_second;
            }
        } else {
            for (;;) {
                __syncthreads();   // everybody is done with the last unit's LDS tiles and has read sh_item
                if (tid == 0) {
                    int vb = -1;
                    for (unsigned k = 0; k < 8 && vb < 0; ++k) {
                        const unsigned x = (xcc + k) & 7u;
                        const int count = (n_vb - (int)x + 7) / 8;   // units x, x + 8, ... below n_vb
                        // (a look before the draw keeps the counters of exhausted lists from running on)
                        if (__hip_atomic_load(pf_drawn + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= count) continue;
                        const int j = __hip_atomic_fetch_add(pf_drawn + x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (j < count) vb = 8 * j + (int)x;
                    }
                    sh_item = vb;
                }
                __syncthreads();
                const int vb = sh_item;
                if (vb < 0) break;
                const int entry = p.pf_table ? min(vb / p.Hkv, p.pf_table - 1) : 0;
                prefill_unit<HD, 4, true, 1>(p, pf_at, vb, entry, vb - entry * p.Hkv, p.pf_table ? pf_at(2 * p.num_pf + 1 + entry) : 0);
                if (pass == 0) ++n_first; else ++n_second;
            }
        }
        __syncthreads();   // the whole workgroup changes its kind of work together
        if (trace && tid == 0) trace[1 + pass] = wall_clock64();
    }
    if (trace && tid == 0) trace[3] += (n_first << 8) + (n_second << 32);
    // leave; the last workgroup out clears the state
    if (tid == 0) {
        const int gone = __hip_atomic_fetch_add(left, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_item = gone == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (sh_item) {
        for (int i = tid; i < kMixedStateInts - 1; i += kPfThreads)
            __hip_atomic_store(state + i, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ------------------------------------------------------------------------------------------
// KV block copy: workgroup (pair, which pool, slice) moves a contiguous slice of one block with
// 16-byte loads and stores; all loads of a thread are issued before its stores.
constexpr int kCopyThreads = 256;

template <int VPT, bool NT>
__global__ __launch_bounds__(kCopyThreads) void block_copy_kernel(const u32x4 *k_src, const u32x4 *v_src, u32x4 *k_dst,
                                                                  u32x4 *v_dst, const int64_t *src_ids,
                                                                  const int64_t *dst_ids, int64_t block_vecs,
                                                                  int slices)
{
    const int64_t pair = blockIdx.x / (2 * slices);
    const int rem = blockIdx.x - pair * (2 * slices);
    const int which = rem / slices;
    const int slice = rem - which * slices;
    const int64_t sb = src_ids[pair], db = dst_ids[pair];
    const u32x4 *src = (which ? v_src : k_src) + sb * block_vecs;
    u32x4 *dst = (which ? v_dst : k_dst) + db * block_vecs;
    const int64_t base = (int64_t)slice * kCopyThreads * VPT + threadIdx.x;
    u32x4 r[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int64_t idx = base + (int64_t)i * kCopyThreads;
        if (idx < block_vecs) r[i] = NT ? __builtin_nontemporal_load(src + idx) : src[idx];
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int64_t idx = base + (int64_t)i * kCopyThreads;
        if (idx < block_vecs) {
            if (NT)
                __builtin_nontemporal_store(r[i], dst + idx);
            else
                dst[idx] = r[i];
        }
    }
}

// ------------------------------------------------------------------------------------------
// KV append: the K and V vectors of the step's tokens go into their paged slots.  One workgroup of 256 threads per
// (sequence, KV block that the step's rows of that sequence touch): the rows of a block are written together, so
// that whole lines leave the compute unit -- K keeps [hd/8][16 slots][8]: the 16-byte pieces of up to 16 rows are
// contiguous per group of 8 dims; V keeps [dim][16 slots]: a thread gathers one (kv head, dim) element from all
// rows of the block and writes them side by side (two 16-byte stores when the step covers the whole block, 2-byte
// stores otherwise).
// Workgroup w -> (sequence, block) without a plan: sequence i owns the workgroup indices [G(i), G(i+1)) with
// G(i) = query_start_loc[i] / 16 + 2 i, which is at least as many as the blocks its q_len rows can touch
// (q_len / 16 + 2); the grid has total_q / 16 + 2 num_seqs + 1 workgroups and those beyond a sequence's last
// block leave at once.  Every workgroup finds its sequence with one 64-lane look at query_start_loc.
constexpr int kAppendThreads = 256;
template <bool PAST>   // 16-byte stores past the caches
OOCO_DEV void kv_append_body(const uint16_t *k_new, const uint16_t *v_new, uint16_t *k_cache, uint16_t *v_cache, const int32_t *block_tables,
                             const int32_t *query_start_loc, const int32_t *ctx_lens, int num_seqs, int total_q, int Hkv, int hd,
                             int max_blocks_per_seq, int64_t num_blocks, int parts, int by_rows)
{
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    // `parts` workgroups share a (sequence, block) pair: each takes every parts-th slice of the rows' elements, so that a pair whose rows cover its block only partly (many narrow stores) does not end last
    const int w = blockIdx.x / parts;
    const int part = blockIdx.x - w * parts;
    // first pair of a sequence, by where its rows start: with `by_rows` it owns a pair per row (rows never touch more blocks)
    auto g_of = [&](int start, int idx) -> int { return by_rows ? start : start / kBlockSize + 2 * idx; };
    auto g_at = [&](int idx) -> int { return g_of(query_start_loc[idx], idx); };
    int seq, q0, q_len, ctx;
    if (num_seqs <= 4 * 64) {
        // up to 256 sequences: the four 64-lane looks are independent loads (one memory round trip), where
        // count_le would wait for each before starting the next; the same round trip brings the lengths of all
        // sequences (lane l of look p holds query_start_loc[64p + l + 1] and ctx_lens[64p + l]), so that the found
        // sequence's own values are a lane read away instead of a second round trip
        int cnt = 0, qv[4], cv[4];
        const int qs0 = query_start_loc[0];   // (0 by the arrays' contract; read in the same round trip all the same)
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int idx = 1 + 64 * pass + lane;
            qv[pass] = idx <= num_seqs ? query_start_loc[idx] : 0x7FFFFFFF;
            cv[pass] = idx <= num_seqs ? ctx_lens[idx - 1] : 0;
        }
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int idx = 1 + 64 * pass + lane;
            const int v = idx <= num_seqs ? g_of(qv[pass], idx) : 0x7FFFFFFF;
            cnt += __popcll(__ballot(v <= w));
        }
        seq = __builtin_amdgcn_readfirstlane(min(cnt, num_seqs - 1));
        // query_start_loc[seq + 1] and ctx_lens[seq] sit in lane seq % 64 of look seq / 64, query_start_loc[seq] in
        // the lane before
        auto pick = [&](const int (&r)[4], int i) -> int {   // value of flat index i (wave-uniform) of a 4 x 64 array
            const int p4 = i >> 6, l = i & 63;
            const int x = p4 == 0 ? r[0] : p4 == 1 ? r[1] : p4 == 2 ? r[2] : r[3];
            return __builtin_amdgcn_readlane(x, l);
        };
        const int q1 = pick(qv, seq);
        q0 = seq > 0 ? pick(qv, seq - 1) : qs0;
        q_len = q1 - q0;
        ctx = pick(cv, seq);
    } else {
        seq = count_le(g_at, num_seqs, w, lane);
        seq = __builtin_amdgcn_readfirstlane(min(seq, num_seqs - 1));
        q0 = query_start_loc[seq];
        q_len = query_start_loc[seq + 1] - q0;
        ctx = ctx_lens[seq];
    }
    if (q_len <= 0 || ctx < 0 || q0 < 0 || q0 + q_len > total_q) return;   // nothing to write / inconsistent arrays
    const int j = w - g_of(q0, seq);          // which of the touched blocks
    const int bidx = ctx / kBlockSize + j;
    if (j < 0 || bidx > (ctx + q_len - 1) / kBlockSize) return;   // beyond the sequence's last touched block
    if (bidx >= max_blocks_per_seq) return;                 // beyond the block table: nothing is written
    // (the id is checked where the stores are, so that the loads of the new vectors do not wait for it)
    const int64_t blk_raw = block_tables[(int64_t)seq * max_blocks_per_seq + bidx];
    const bool blk_ok = blk_raw >= 0 && blk_raw < num_blocks;   // id outside the pool: nothing is written
    const int64_t blk = blk_ok ? blk_raw : 0;
    // rows t_lo .. t_lo + nrow - 1 of the sequence fall into this block, starting at slot slot0
    const int t_lo = max(0, bidx * kBlockSize - ctx);
    const int slot0 = ctx + t_lo - bidx * kBlockSize;
    const int nrow = min(kBlockSize - slot0, q_len - t_lo);
    const int row_elems = Hkv * hd, chunks = row_elems / 8;
    const int64_t row0 = (int64_t)(q0 + t_lo);
    const uint16_t *const k_src = k_new + row0 * row_elems, *const v_src = v_new + row0 * row_elems;
    u32x4 *const k_dst = reinterpret_cast<u32x4 *>(k_cache) + (int64_t)blk * chunks * kBlockSize + slot0;
    uint16_t *const v_dst = v_cache + (int64_t)blk * row_elems * kBlockSize;   // slot 0 of the first cache row
    // (the 2-byte stores of a decode row's V lose past the caches: 64 decodes 4.4 -> 5.5 us)
    auto store16 = [](const u32x4 &v, u32x4 *d) {
        if constexpr (PAST)
            __builtin_nontemporal_store(v, d);
        else
            *d = v;
    };
    if (nrow == kBlockSize) {   // a whole block
        // K: thread -> (row r = tid % 16, 16-byte chunk c = tid / 16 + 16 i): the 16 rows of a chunk are adjacent in
        // the cache, so a wave's stores cover 4 chunks x 256 contiguous bytes
        const u32x4 *src = reinterpret_cast<const u32x4 *>(k_src + (int64_t)(tid & 15) * row_elems);
        u32x4 *dst = k_dst + (tid & 15);
        constexpr int kSlice = kAppendThreads / 16;   // chunks a workgroup moves per pass
        for (int c0 = (tid >> 4) + kSlice * part; c0 < chunks; c0 += 2 * kSlice * parts) {
            u32x4 v[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int c = c0 + i * kSlice * parts;
                if (c < chunks) v[i] = src[c];
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int c = c0 + i * kSlice * parts;
                if (c < chunks && blk_ok) store16(v[i], &dst[(int64_t)c * kBlockSize]);
            }
        }
        // V: thread -> element e = (kv head, dim) of all rows, 32 contiguous bytes of the cache.  (Two adjacent elements
        // per thread, or all loads of a workgroup before its first store, are slower here: 8 x 512 rows and 128 decodes
        // 11.1 -> 12.3 and 12.5 us.)
        for (int e = tid + kAppendThreads * part; e < row_elems; e += kAppendThreads * parts) {
            const uint16_t *s = v_src + e;
            uint32_t x[8];
#pragma unroll
            for (int r = 0; r < 8; ++r)
                x[r] = (uint32_t)s[(int64_t)(2 * r) * row_elems] | ((uint32_t)s[(int64_t)(2 * r + 1) * row_elems] << 16);
            u32x4 *d4 = reinterpret_cast<u32x4 *>(v_dst + (int64_t)e * kBlockSize);
            if (blk_ok) {
                store16(u32x4{x[0], x[1], x[2], x[3]}, d4);
                store16(u32x4{x[4], x[5], x[6], x[7]}, d4 + 1);
            }
        }
        return;
    }
    // A block that the step covers partly -- a decode row, the ends of a chunk --: few bytes, so what counts is the
    // number of memory round trips, and a pass over the elements of every row sends off all its loads, of K and of V,
    // before its first store (128 decodes 6.5 -> 5.6 us, 512 15.7 -> 12.9).  K as above; V: E adjacent elements per
    // thread, x[s] = their values in slot s of the block.  Two elements, or one for rows that two would leave half the
    // threads without (4 heads of 64, six chunks of 3..14 rows: 4.6 us, with two 5.1).
    const bool v_aligned = ((uintptr_t)v_new & 3) == 0;   // (rows have an even number of elements)
    auto partly = [&](auto per_thread) {
        constexpr int E = decltype(per_thread)::value, PASS = E * kAppendThreads;
        for (int e0 = PASS * part; e0 < row_elems; e0 += PASS * parts) {
            constexpr int KI = PASS / 8 / (kAppendThreads / 16);
            const int r = tid & 15, c0 = e0 / 8 + (tid >> 4), e = e0 + E * tid;
            u32x4 kv[KI];
#pragma unroll
            for (int i = 0; i < KI; ++i)
                if (r < nrow && c0 + 16 * i < chunks)
                    kv[i] = reinterpret_cast<const u32x4 *>(k_src + (int64_t)r * row_elems)[c0 + 16 * i];
            uint32_t x[kBlockSize];
            if (e < row_elems) {
#pragma unroll
                for (int sl = 0; sl < kBlockSize; ++sl) {
                    const uint16_t *const src = v_src + (int64_t)(sl - slot0) * row_elems + e;
                    x[sl] = 0;
                    if (sl >= slot0 && sl < slot0 + nrow)
                        x[sl] = E == 1 ? (uint32_t)src[0]
                                : v_aligned ? *reinterpret_cast<const uint32_t *>(src) : (uint32_t)src[0] | ((uint32_t)src[1] << 16);
                }
            }
            if (!blk_ok) continue;
#pragma unroll
            for (int i = 0; i < KI; ++i)
                if (r < nrow && c0 + 16 * i < chunks) store16(kv[i], &k_dst[(int64_t)(c0 + 16 * i) * kBlockSize + r]);
            if (e < row_elems) {
                // quarters of a cache row (4 slots = 8 bytes) that the step covers whole are written with one store
                // each, the ragged ends slot by slot
#pragma unroll
                for (int h = 0; h < E; ++h) {
                    uint16_t *const row = v_dst + (int64_t)(e + h) * kBlockSize;   // (32-byte aligned)
                    auto at = [&](int sl) -> uint32_t { return h ? x[sl] >> 16 : x[sl] & 0xFFFFu; };
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (4 * q >= slot0 && 4 * q + 4 <= slot0 + nrow) {
                            *reinterpret_cast<u32x2 *>(row + 4 * q) =
                                u32x2{at(4 * q) | (at(4 * q + 1) << 16), at(4 * q + 2) | (at(4 * q + 3) << 16)};
                        } else {
#pragma unroll
                            for (int sl = 4 * q; sl < 4 * q + 4; ++sl)
                                if (sl >= slot0 && sl < slot0 + nrow) row[sl] = (uint16_t)at(sl);
                        }
                    }
                }
            }
        }
    };
    if (row_elems >= 2 * kAppendThreads)
        partly(std::integral_constant<int, 2>());
    else
        partly(std::integral_constant<int, 1>());
}
__global__ __launch_bounds__(kAppendThreads) void kv_append_kernel(const uint16_t *k_new, const uint16_t *v_new, uint16_t *k_cache, uint16_t *v_cache,
                                                                   const int32_t *block_tables, const int32_t *query_start_loc,
                                                                   const int32_t *ctx_lens, int num_seqs, int total_q, int Hkv, int hd,
                                                                   int max_blocks_per_seq, int64_t num_blocks, int parts, int by_rows)
{
    kv_append_body<true>(k_new, v_new, k_cache, v_cache, block_tables, query_start_loc, ctx_lens, num_seqs, total_q, Hkv, hd, max_blocks_per_seq,
                         num_blocks, parts, by_rows);
}
__global__ __launch_bounds__(kAppendThreads) void kv_append_kernel_cached(const uint16_t *k_new, const uint16_t *v_new, uint16_t *k_cache,
                                                                          uint16_t *v_cache, const int32_t *block_tables,
                                                                          const int32_t *query_start_loc, const int32_t *ctx_lens, int num_seqs,
                                                                          int total_q, int Hkv, int hd, int max_blocks_per_seq,
                                                                          int64_t num_blocks, int parts, int by_rows)
{
    kv_append_body<false>(k_new, v_new, k_cache, v_cache, block_tables, query_start_loc, ctx_lens, num_seqs, total_q, Hkv, hd, max_blocks_per_seq,
                          num_blocks, parts, by_rows);
}

hipError_t launch_kv_append(const void *k_new, const void *v_new, void *k_cache, void *v_cache, const int32_t *block_tables,
                            const int32_t *query_start_loc, const int32_t *ctx_lens, int num_seqs, int total_q, int Hkv,
                            int hd, int max_blocks_per_seq, int64_t num_blocks, int parts_opt, int num_cus, hipStream_t s)
{
    if (total_q <= 0 || num_seqs <= 0) return hipSuccess;
    // One workgroup per 512 elements of a row.  8 kv heads x 128, 4,224 tokens, 1 / 2 / 4 / 8 parts: 12.7 / 10.4 / 13.1 /
    // 16.5 us; 32 x 128, 16 decodes: 18.2 / 10.2 / 6.6 / 4.7, 4096 chunk rows: 61 / 41 / 36 / 32.
    const int parts = parts_opt > 0 ? std::min(parts_opt, 8) : std::max(1, std::min(8, Hkv * hd / (2 * kAppendThreads)));
    // Workgroups without a block to write cost their start all the same.  A sequence owns two (sequence, block) pairs and one more per
    // 16 rows before its end, twice what a batch of decode rows needs; where nearly all sequences have one row, and the pairs are
    // more than one per compute unit, it owns a pair per row.  MI355X (us): 200 decodes, 8 kv heads of 128 7.18 -> 6.34, 400 of 4
    // heads 7.39 -> 6.62, 150 of 8 heads of 64 5.25 -> 4.60, 64 of 8 heads of 128 level; 91 of 4 heads, under 256 pairs, 5.14 -> 5.23.
    const int64_t pairs = total_q / kBlockSize + 2 * (int64_t)num_seqs + 1;
    const bool by_rows = append_by_rows(total_q, num_seqs, pairs * parts, num_cus);
    const unsigned grid = (unsigned)((by_rows ? total_q : pairs) * parts);
    // Attention reads what was appended next.  A few prompts' keys are all that it reads for a while, and it finds them in the caches
    // unless they went past them; many decode rows, or a prefill part beside them, are faster out of the way of the old keys, and so
    // is whatever is more than the caches keep.  Append and attention of a captured layer, MI355X (us), through the caches / past them:
    // 1000 rows 27.0 / 28.4, prompts of 1000, 700 and 300 30.1 / 32.0, 1000 rows beside 8 / 16 / 32 decodes 26.9 / 29.4, 38.2 / 37.5,
    // 58.9 / 57.2, 8 x 512 beside 128 287.6 / 279.7, 64 decodes 82.2 / 80.9, 200 160.3 / 154.7, 8 x 512 and 2 x 2048 rows level.  The
    // append alone: 5 rows and 3 decodes 6.4 / 6.6, 1000 rows 6.2 / 5.8, 8 x 512 10.0 / 9.4, with 128 decodes 12.3 / 10.9.
    const bool past = append_past_caches(total_q, num_seqs, 4 * (int64_t)total_q * Hkv * hd);
    hipLaunchKernelGGL(past ? kv_append_kernel : kv_append_kernel_cached, dim3(grid), dim3(kAppendThreads), 0, s, (const uint16_t *)k_new,
                       (const uint16_t *)v_new, (uint16_t *)k_cache, (uint16_t *)v_cache, block_tables, query_start_loc,
                       ctx_lens, num_seqs, total_q, Hkv, hd, max_blocks_per_seq, num_blocks, parts, (int)by_rows);
    return hipGetLastError();
}


// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fill_zero_kernel(int32_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_fill_zero(int32_t *p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_decode(const KernArgs &a, hipStream_t s)
{
    if (a.p.static_runs <= 0 || a.p.dec_blocks <= 0) return hipSuccess;
    const dim3 grid((unsigned)((int64_t)a.p.static_runs * a.p.Hkv)), block(64);
    if (a.p.coop) {
        if (a.p.coop_waves == 8) {   // (planned for batches whose arrays fit the arguments only)
            if (a.p.cum_dev) return hipErrorInvalidValue;
            if (a.p.hd == 128)
                hipLaunchKernelGGL((decode_coop_kernel_groups<128, 2>), grid, dim3(512), 0, s, a);
            else
                hipLaunchKernelGGL((decode_coop_kernel_groups<64, 4>), grid, dim3(512), 0, s, a);
        } else if (a.p.cum_dev) {
            if (a.p.hd == 128)
                hipLaunchKernelGGL((decode_coop_kernel_general<128, 2>), grid, dim3(256), 0, s, a);
            else
                hipLaunchKernelGGL((decode_coop_kernel_general<64, 4>), grid, dim3(256), 0, s, a);
        } else if (a.p.hd == 128) {
            hipLaunchKernelGGL((decode_coop_kernel<128, 2>), grid, dim3(256), 0, s, a);
        } else {
            hipLaunchKernelGGL((decode_coop_kernel<64, 4>), grid, dim3(256), 0, s, a);
        }
        return hipGetLastError();
    }
    const bool general = a.p.tail_runs > 0 || a.p.xcd_cw[kXcds - 1] != 0 || a.p.cum_dev;
    if (a.p.lean && a.p.hd == 128) {
        if (general)
            hipLaunchKernelGGL((decode_kernel_lean_general<128>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((decode_kernel_lean<128>), grid, block, 0, s, a);
        return hipGetLastError();
    }
    // KV blocks per softmax step: a wave keeps one step's tiles in flight, and 8 KiB per wave is what it takes
    // to saturate HBM with three waves per compute unit: one block for head_dim 128, two for head_dim 64
    // (measured: 56.9 % -> 72.2 % of the HBM peak on 256 sequences with head_dim 64; four blocks: 69.8 %)
    const int nbi = a.p.nbi ? a.p.nbi : (a.p.hd == 64 ? 2 : 1);
    if (general) {
        if (a.p.hd == 128) {
            if (nbi == 2)
                hipLaunchKernelGGL((decode_kernel_general<128, 2>), grid, block, 0, s, a);
            else if (nbi == 4)
                hipLaunchKernelGGL((decode_kernel_general<128, 4>), grid, block, 0, s, a);
            else
                hipLaunchKernelGGL((decode_kernel_general<128, 1>), grid, block, 0, s, a);
        } else {
            if (nbi == 2)
                hipLaunchKernelGGL((decode_kernel_general<64, 2>), grid, block, 0, s, a);
            else if (nbi == 4)
                hipLaunchKernelGGL((decode_kernel_general<64, 4>), grid, block, 0, s, a);
            else
                hipLaunchKernelGGL((decode_kernel_general<64, 1>), grid, block, 0, s, a);
        }
        return hipGetLastError();
    }
    if (a.p.hd == 128) {
        if (nbi == 2)
            hipLaunchKernelGGL((decode_kernel<128, 2>), grid, block, 0, s, a);
        else if (nbi == 4)
            hipLaunchKernelGGL((decode_kernel<128, 4>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((decode_kernel<128, 1>), grid, block, 0, s, a);
    } else {
        if (nbi == 2)
            hipLaunchKernelGGL((decode_kernel<64, 2>), grid, block, 0, s, a);
        else if (nbi == 4)
            hipLaunchKernelGGL((decode_kernel<64, 4>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((decode_kernel<64, 1>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_prefill(const KernArgs &a, hipStream_t s)
{
    if (a.p.n_tiles <= 0) return hipSuccess;
    const dim3 grid = a.p.pf_table ? dim3((unsigned)a.p.Hkv, (unsigned)a.p.pf_table)
                                   : dim3((unsigned)((int64_t)a.p.n_tiles * a.p.Hkv * (a.p.pf_split > 0 ? a.p.pf_split : 1)));
    if (a.p.pf_groups > 1 && a.p.hd == 128)
        hipLaunchKernelGGL((prefill_kernel_groups<128>), grid, dim3(512), 0, s, a);
    else if (a.p.pf_groups > 1)
        hipLaunchKernelGGL((prefill_kernel_groups<64>), grid, dim3(512), 0, s, a);
    else if (a.p.hd == 128 && a.p.pf_waves == 8 && a.p.lean)
        hipLaunchKernelGGL((prefill_kernel_lean<128>), grid, dim3(512), 0, s, a);
    else if (a.p.hd == 128 && a.p.pf_waves == 8)
        hipLaunchKernelGGL((prefill_kernel<128, 8>), grid, dim3(512), 0, s, a);
    else if (a.p.hd == 128)
        hipLaunchKernelGGL((prefill_kernel<128, 4>), grid, dim3(kPfThreads), 0, s, a);
    else
        hipLaunchKernelGGL((prefill_kernel<64, 4>), grid, dim3(kPfThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_step(KernArgs &a, int num_cus, hipStream_t s)
{
    if (a.p.n_tiles <= 0 || a.p.static_runs <= 0 || a.p.cum_dev || a.p.tail_runs > 0) return hipErrorInvalidValue;
    // Decode waves of a workgroup: as few as put a decode workgroup on every unit, at most one per SIMD.  (24 sequences,
    // 384 waves: four to a workgroup the stream has the vector-memory paths of 96 units only)
    const int64_t items = (int64_t)a.p.static_runs * a.p.Hkv;
    a.p.dec_wpw = a.p.coop ? 1 : (int8_t)std::min<int64_t>(kStepDecWaves, (items + num_cus - 1) / num_cus);
    const int64_t dec = (items + a.p.dec_wpw - 1) / a.p.dec_wpw;
    const int64_t pf = a.p.pf_table ? (int64_t)a.p.pf_table * a.p.Hkv
                                    : (int64_t)a.p.n_tiles * a.p.Hkv * (a.p.pf_split > 0 ? a.p.pf_split : 1);
    a.p.dec_wgs = (int32_t)dec;
    if (dec + pf > 2 * (int64_t)num_cus) a.p.pf_share = 0;   // (two workgroups of four waves fit a unit, of either head_dim)
    // rows: the decode runs of cooperative workgroups, then the tile list's entries
    if (a.p.rows2d && (!a.p.coop || !a.p.pf_table || a.p.list_row != a.p.static_runs)) return hipErrorInvalidValue;
    const dim3 grid = a.p.rows2d ? dim3((unsigned)a.p.Hkv, (unsigned)(a.p.static_runs + a.p.pf_table)) : dim3((unsigned)(dec + pf));
    if (a.p.pf_groups > 1 && (!a.p.coop || a.p.coop_waves != 8)) return hipErrorInvalidValue;
    if (a.p.pf_groups > 1 && a.p.hd == 128)
        hipLaunchKernelGGL((step_kernel_groups<128, 2>), grid, dim3(512), 0, s, a);
    else if (a.p.pf_groups > 1)
        hipLaunchKernelGGL((step_kernel_groups<64, 4>), grid, dim3(512), 0, s, a);
    else if (a.p.lean)
        hipLaunchKernelGGL((step_kernel_lean<128>), grid, dim3(512), 0, s, a);
    else if (a.p.hd == 64 && a.p.coop)
        hipLaunchKernelGGL((step_kernel<64, 4, true>), grid, dim3(kPfThreads), 0, s, a);
    else if (a.p.hd == 64)
        hipLaunchKernelGGL((step_kernel<64, 2, false>), grid, dim3(kPfThreads), 0, s, a);
    else if (a.p.coop)
        hipLaunchKernelGGL((step_kernel<128, 2, true>), grid, dim3(kPfThreads), 0, s, a);
    else if (a.p.nbi == 2)
        hipLaunchKernelGGL((step_kernel<128, 2, false>), grid, dim3(kPfThreads), 0, s, a);
    else
        hipLaunchKernelGGL((step_kernel<128, 1, false>), grid, dim3(kPfThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_mixed(const KernArgs &a, int num_cus, hipStream_t s)
{
    if (a.p.n_tiles <= 0 || a.p.static_runs <= 0) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(2 * num_cus)), block(kPfThreads);
    if (a.p.hd == 128)
        hipLaunchKernelGGL((mixed_kernel<128>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((mixed_kernel<64>), grid, block, 0, s, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// The pairs of a block copy in order of the region of the destination pool they go to (see ooco_sort.hip for why the
// order matters): a counting sort by the leading bits of the destination id, one workgroup, one launch.  What the copy
// needs is that the few hundred blocks written at a time are neighbours, so pairs of one bucket stay in any order, and a
// full sort by all bits (the library's radix sort, five launches, 28 us for 11,000 pairs) buys nothing more.  Bound by
// latency -- load the ids, count, scan, write --, so the ids stay in registers between the passes, the pairs are put in
// order in LDS (8-byte stores scattered over memory by one unit would cost more than all the rest) and written out in
// whole lines.  Whatever the ids, the result is a permutation of the pairs (ids of blocks fit 31 bits).
constexpr int kOrderThreads = 1024, kOrderBuckets = 4096;
__global__ __launch_bounds__(kOrderThreads) void order_pairs_kernel(const int64_t *dst_ids, const int64_t *src_ids,
                                                                    int64_t *dst_out, int64_t *src_out, int num_pairs,
                                                                    int shift)
{
    constexpr int U = (int)(kOrderPairsMax / kOrderThreads), PER = kOrderBuckets / kOrderThreads;
    static_assert(U * kOrderThreads == kOrderPairsMax, "whole passes");
    __shared__ u32x2 pairs[kOrderPairsMax];
    __shared__ int start[kOrderBuckets];
    __shared__ int wave_sum[kOrderThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t d[U], s[U];
    int rank[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min(u * kOrderThreads + tid, num_pairs - 1);
        if (u * kOrderThreads < num_pairs) {
            d[u] = (uint32_t)dst_ids[i];
            s[u] = (uint32_t)src_ids[i];
        }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) start[i * kOrderThreads + tid] = 0;
    __syncthreads();
    auto bucket = [&](uint32_t id) -> int { return (int)((id >> shift) & (uint32_t)(kOrderBuckets - 1)); };
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u * kOrderThreads + tid < num_pairs) rank[u] = atomicAdd(&start[bucket(d[u])], 1);
    __syncthreads();
    // exclusive scan: PER buckets a thread, then the waves, then the workgroup
    int c[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = sum;
        sum += start[tid * PER + i];
    }
    int incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int before = incl - sum;
#pragma unroll
    for (int w = 0; w < kOrderThreads / 64; ++w) before += w < wave ? wave_sum[w] : 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) start[tid * PER + i] = before + c[i];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (u * kOrderThreads + tid < num_pairs) pairs[start[bucket(d[u])] + rank[u]] = u32x2{d[u], s[u]};
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = u * kOrderThreads + tid;
        if (i < num_pairs) {
            const u32x2 x = pairs[i];
            dst_out[i] = (int64_t)x[0];
            src_out[i] = (int64_t)x[1];
        }
    }
}

hipError_t launch_order_pairs(const int64_t *dst_ids, int64_t *dst_out, const int64_t *src_ids, int64_t *src_out,
                              int64_t num_pairs, int bits, hipStream_t s)
{
    int shift = 0;
    while (((int64_t)kOrderBuckets << shift) < ((int64_t)1 << bits)) ++shift;
    hipLaunchKernelGGL(order_pairs_kernel, dim3(1), dim3(kOrderThreads), 0, s, dst_ids, src_ids, dst_out, src_out, (int)num_pairs,
                       shift);
    return hipGetLastError();
}

hipError_t launch_block_copy(const void *k_src, const void *v_src, void *k_dst, void *v_dst, const int64_t *src_ids,
                             const int64_t *dst_ids, int64_t num_pairs, int64_t block_bytes, int variant, hipStream_t s)
{
    if (num_pairs == 0) return hipSuccess;
    const int64_t block_vecs = block_bytes / 16;
    if (variant == 0) variant = 41;
    const int vpt = variant / 10;
    const int per_wg = kCopyThreads * vpt;
    const int slices = (int)((block_vecs + per_wg - 1) / per_wg);
    const dim3 grid((unsigned)(num_pairs * 2 * slices)), block(kCopyThreads);
#define OOCO_COPY(V, N)                                                                                              \
    hipLaunchKernelGGL((block_copy_kernel<V, N>), grid, block, 0, s, (const u32x4 *)k_src, (const u32x4 *)v_src,      \
                       (u32x4 *)k_dst, (u32x4 *)v_dst, src_ids, dst_ids, block_vecs, slices)
    switch (variant) {
    case 20: OOCO_COPY(2, false); break;
    case 21: OOCO_COPY(2, true); break;
    case 40: OOCO_COPY(4, false); break;
    case 80: OOCO_COPY(8, false); break;
    case 81: OOCO_COPY(8, true); break;
    case 10: OOCO_COPY(1, false); break;
    case 11: OOCO_COPY(1, true); break;
    default: OOCO_COPY(4, true); break;
    }
#undef OOCO_COPY
    return hipGetLastError();
}

}  // namespace ooco
