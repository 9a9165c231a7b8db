// Packed prefill attention, bf16 MFMA, head dimension PK_D = 128 or 64 (Sec. 3.1).  Same tables and
// arithmetic as prefill.hip (S^T = K.Q^T, O^T += V^T.P^T, one wave per 32 query rows, key tiles of 64), but
//   * K/V tiles go HBM/L2 -> LDS directly (buffer_load ... lds, 16 bytes per lane, no staging
//     registers, hardware bounds check) into slabs of 64 columns; the 16-byte chunks of a row are
//     XOR-swizzled -- the swizzle is applied on the global side of the copy, so that both the K
//     row reads (ds_read_b128) and the V transpose reads (ds_read_b64_tr_b16) are free of bank
//     conflicts;
//   * a key tile is processed as two halves of 32 keys, in a software pipeline: the softmax of one half is dealt
//     over the MFMAs that make the scores of the next half but one and those that take the probabilities of the half
//     before, and the LDS operand reads run four steps ahead in a ring of registers: matrix pipe,
//     vector ALU and LDS overlap inside one wave;
//   * the MFMA is v_mfma_f32_16x16x32_bf16.  Under this load the clock is managed by power, and per flop the 32x32x16
//     form costs more of it (MFMAs alone on random operands: 1.75 PFLOP/s at 1.70 GHz against 2.07 at 2.02).

// Device code only: included by prefill_pipe.hip (the prefill launch) and by mixed_step.hip (the
// fused prefill + decode launch).  The includer defines PK_D (the head dimension), PK_WAVES (4, or 8 for twice the query heads of
// a KV head) and PK_DNS (the namespace this instance goes into) first; the file may be included once per combination.
#include <cstdint>

#include "common.hip.h"
#include "kernels.h"

#if !defined(PK_D) || !defined(PK_DNS) || !defined(PK_WAVES) || (PK_D != 128 && PK_D != 64) || (PK_WAVES != 4 && PK_WAVES != 8)
#error "define PK_D (128 or 64), PK_WAVES (4 or 8) and PK_DNS before including prefill_body.hip.h"
#endif

namespace pk {
namespace {
namespace PK_DNS {

constexpr int BM = 128, BN = 64, D = PK_D;
constexpr int ROWB = D * 2;                        // bytes per K/V row in global memory
constexpr int TILE_BYTES = BN * ROWB;              // 16 KiB (8 KiB for D = 64)
constexpr int KS = D / 32;                         // contraction steps of a score
constexpr int OPS = D / 16;                        // LDS operands per half tile, of K (two blocks of 16 keys x KS) as of V (blocks of 16 columns)
constexpr int NC = 2;                              // column blocks of a wave: block c holds its rows 16 c .. + 15
constexpr int WAVES = PK_WAVES;                     // 4, or 8: twice the heads on the same K/V tiles
constexpr int PIECES = TILE_BYTES / (1024 * WAVES);   // 1-KiB copy instructions per wave and tile
constexpr int RPW = BN / WAVES, PPS = RPW / 8;        // rows (and copies) of a slab that one wave fills

// A stage in LDS is one slab per 64 columns: 64 rows of 128 bytes (eight 16-byte chunks).  Whatever
// the head dimension, two K and four V addresses per lane then reach every operand with constant
// offsets, six additions to the stage's address per key tile.
constexpr int SLAB_ROWB = 128, SLAB = BN * SLAB_ROWB;

typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Chunk position p of row `row` holds logical chunk p ^ swz(row).  Two 128-byte rows share a line of the 64 banks.  A
// 16-byte read (K: rows 0 .. 15, lane group g at chunk g) is served in sets of sixteen lanes, of which one takes rows 0 .. 3 and 12 .. 15
// at an even chunk and rows 4 .. 11 at the odd one next to it: the eight rows of a parity need eight different positions,
// and those of rows 4 .. 11 pairs 2 i, 2 i + 1.  A transpose read (V) takes 32 bytes, two chunks, from each of eight consecutive
// rows per 32 lanes: four rows of a parity need different pairs.
__device__ __forceinline__ int swz(int row) { const int x = (row >> 1) & 7; return (((x & 3) ^ ((x >> 1) & 2)) << 1) | (x >> 2); }

struct LaneOffsets {
    int k[2];           // K operand read: row n, logical chunk 4 (s & 1) + g of a slab
    int v[4];           // V transpose reads of column block t & 3 of a slab: rows 4 g .. + 3 (and 16 behind them)
    int g[PIECES];      // global byte offsets of this lane's copy instructions
};

// A operand of P.V, columns 16 t .. + 15 of V as rows: lane (n, g) holds keys 4 g + j (j < 4) and 16 + 4 g + j - 4 of
// half tile kb, the order in which the scores of its query leave the S MFMAs.
__device__ __forceinline__ bf16x4 v_half_operand(const unsigned char* vs, const LaneOffsets& lo, int kb, int t, int half) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(vs + (t >> 2) * SLAB + (32 * kb + 16 * half) * SLAB_ROWB + lo.v[t & 3]));
}
__device__ __forceinline__ bf16x8 v_operand(const unsigned char* vs, const LaneOffsets& lo, int kb, int t) {
    return __builtin_shufflevector(v_half_operand(vs, lo, kb, t, 0), v_half_operand(vs, lo, kb, t, 1), 0, 1, 2, 3, 4, 5, 6, 7);
}

// What a workgroup works on, and this lane's share of it.
struct WorkUnit {
    int head, kvh, n_kv, n_lead, n_active, wave, lane, n, g;   // this wave's head; it computes key tiles [n_lead, n_active)
    int rows;                          // which 32 of the tile's rows this wave has
    int ks[3], info[3];                // (first key row, info) of the tile's first three key tiles (the last one repeated)
    int qrow[2], lo[2], hi[2];         // this lane's query rows (-1: padding) and their key ranges [lo, hi)
    const int32_t* kvt;                // key-tile list of the query tile: (first key row, info) pairs
    int k_end, full;                   // keys from k_end on are not the tile's; up to `full` all of this wave's rows see them (row_shift < 2)
    int64_t row_bytes;                 // bytes between consecutive K/V rows in global memory
    uint32_t row_bytes32;              // the same in 32 bits
};

// Decodes the workgroup id, loads the row metadata and the Q operand, derives the lane offsets.
// Returns false for grid padding and for query tiles without key tiles.
__device__ __forceinline__ bool setup(const PrefillArgs& a, const int block, WorkUnit& u, LaneOffsets& off, bf16x8 (&qf)[NC][KS]) {
    // Consecutive workgroup ids go round-robin over the 8 XCDs: the workgroups of one (tile, KV head) pair
    // (heads_per_kv of them, each with its share of the KV head's query heads) stay on one XCD and adjacent in time, so that its L2
    // serves their K/V tiles.
    const int y = block >> 3, slot = a.by_r(y), p = slot * 8 + (block & 7);
    const int tile = a.by_hkv(p);
    if (tile >= a.n_tiles) return false;
    u.kvh = p - tile * a.Hkv;
    const int groups = a.heads_per_kv, group = y - slot * groups;
    // everything about the tile in one 64-byte scalar load, including the first key rows of its first
    // key tiles: the first K/V copies do not wait for the key-tile list
    typedef int32_t i32x16 __attribute__((ext_vector_type(16)));
    const i32x16 desc = *(const __attribute__((address_space(4))) i32x16*)(a.tiles + 16 * static_cast<int64_t>(tile));
    u.n_kv = desc[1];
    if (u.n_kv == 0) return false;
    u.kvt = a.kvtiles + 2 * static_cast<int64_t>(desc[0]);
#pragma unroll
    for (int x = 0; x < 3; ++x) { u.ks[x] = desc[8 + x]; u.info[x] = desc[11 + x]; }
    u.k_end = desc[14];
    const int tid = threadIdx.x;
    u.lane = tid & 63; u.n = u.lane & 15; u.g = u.lane >> 4;
    u.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Wave w of every workgroup runs on SIMD w % 4, and the last rows of a causal tile see more key tiles than
    // the first: every other set of 256 workgroups (a set is one per compute unit) deals
    // the rows in reverse, so that the waves of a SIMD get as much together as those of any other.
    const int part = u.wave & ((1 << a.row_shift) - 1), mate = u.wave >> a.row_shift;
    u.head = ((u.kvh * groups + group) << ((WAVES == 8 ? 3 : 2) - a.row_shift)) + mate;
    u.rows = (WAVES > 4 ? mate & 1 : (block >> 8) & 1) ? (1 << a.row_shift) - 1 - part : part;
    u.n_active = u.n_kv - ((desc[3] >> (8 * u.rows)) & 0xFF);
    u.n_lead = min((desc[2] >> (8 * u.rows)) & 0xFF, u.n_active);
#pragma unroll
    for (int c = 0; c < 2; ++c)
        prefill_tile_row(a, tile, desc[4], desc[5], desc[6], desc[7], u.rows * 32 + 16 * c + u.n, u.qrow[c], u.lo[c], u.hi[c]);
    u.full = a.row_shift < 2 ? __builtin_amdgcn_readfirstlane(u.hi[0]) : 0x7FFFFFFF;   // (the first row's; what one row sees, those behind it do)
    u.row_bytes = static_cast<int64_t>(a.Hkv) * ROWB;
    u.row_bytes32 = static_cast<uint32_t>(a.Hkv) * ROWB;

#pragma unroll
    for (int s = 0; s < 2; ++s) off.k[s] = u.n * SLAB_ROWB + (((4 * s + u.g) ^ swz(u.n)) << 4);
    const int row = 4 * u.g + (u.n >> 2);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        off.v[t] = row * SLAB_ROWB + (((2 * t + ((u.n & 3) >> 1)) ^ swz(row)) << 4) + (u.n & 1) * 8;
    const int r_in = u.lane >> 3, pos = u.lane & 7;    // a copy instruction takes 8 rows of 8 chunks
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int crow = RPW * u.wave + 8 * (q % PPS) + r_in;
        off.g[q] = static_cast<int>(crow * u.row_bytes + u.kvh * ROWB + (q / PPS) * SLAB_ROWB + ((pos ^ swz(crow)) << 4));
    }
    // Q operand: lane (n, g) holds Q[row n of block c][32s + 8g .. +8], as it is in memory: the MFMAs
    // deliver raw scores, exact products of the bf16 inputs summed in fp32.  Only requested here;
    // the first K copies follow at once, so that the two round trips to memory overlap.  Lanes without
    // a query read row 0 and are cleared once it is there (clear_absent_rows).
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int qrow = u.qrow[c];
        const uint16_t* qp = static_cast<const uint16_t*>(a.q) +
                             (static_cast<int64_t>(qrow < 0 ? 0 : qrow) * a.Hq + u.head) * D + 8 * u.g;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[c][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qp + 32 * s));
    }
    return true;
}

// Zeros for the lanes without a query: row 0, which they have read, is another request's and may hold anything.
__device__ __forceinline__ void clear_absent_rows(const WorkUnit& u, bf16x8 (&qf)[NC][KS]) {
    if (__builtin_amdgcn_ballot_w64(u.qrow[0] < 0 || u.qrow[1] < 0) == 0) return;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const u32x4 raw = __builtin_bit_cast(u32x4, qf[c][s]);
            qf[c][s] = __builtin_bit_cast(bf16x8, u.qrow[c] < 0 ? u32x4{0u, 0u, 0u, 0u} : raw);
        }
}

// 1 / row sum (0 for a row without a visible key)
__device__ __forceinline__ float row_scale(const float l) { return l == 0.f ? 0.f : 1.f / l; }

// o / l of head `h` to global memory; lane (n, g) owns columns 16t + 4g .. +3 of its two query rows.
__device__ __forceinline__ void store_output(const PrefillArgs& a, const WorkUnit& u, const floatx4 (&o)[NC][OPS], const floatx4 (&l)[NC]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float inv = row_scale(l[c][0]);
        if (u.qrow[c] < 0) continue;
        float* out = static_cast<float*>(a.out) + (static_cast<int64_t>(u.qrow[c]) * a.Hq + u.head) * D + 4 * u.g;
#pragma unroll
        for (int t = 0; t < OPS; ++t) {
            const floatx4 x = o[c][t];
            *reinterpret_cast<float4*>(out + 16 * t) = make_float4(x[0] * inv, x[1] * inv, x[2] * inv, x[3] * inv);
        }
    }
}

// The same in bf16.  Of two neighbouring blocks of 16 columns the lane groups 1 and 3 give away the first and the groups 0 and 2 the
// second: every lane then has 16 contiguous bytes, a store instruction writes 64 from each of 16 rows, and nothing
// goes through LDS (there the rows leave whole, but the round trip, a look-up of every row and the branches around eight stores
// take 3200 cycles of a workgroup, this 1200: 64 ragged prompts 377.2 -> 373.3 us, 8 x 2048 286.9 -> 283.7, with head dimension 64
// 162.2 -> 160.8, 1 x 4096 with 64 heads 241.3 -> 236.9; short lists in launches of 70 us the same).
__device__ __forceinline__ void store_output_bf16(const PrefillArgs& a, const WorkUnit& u, const floatx4 (&o)[NC][OPS], const floatx4 (&l)[NC]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const float inv = row_scale(l[c][0]);
        if (u.qrow[c] < 0) continue;
        uint16_t* out = static_cast<uint16_t*>(a.out) + (static_cast<int64_t>(u.qrow[c]) * a.Hq + u.head) * D + 16 * (u.g & 1) + 8 * (u.g >> 1);
#pragma unroll
        for (int t = 0; t < OPS; t += 2) {
            uint32_t w[2][2];                          // [block t, t + 1][columns 4g, 4g + 1 / + 2, + 3]
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const floatx4 x = o[c][t + b];
                w[b][0] = pack_bf16x2(x[0] * inv, x[1] * inv); w[b][1] = pack_bf16x2(x[2] * inv, x[3] * inv);
            }
            const auto p0 = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
            const auto p1 = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
            *reinterpret_cast<u32x4*>(out + 16 * t) = u32x4{p0[0], p1[0], p0[1], p1[1]};
        }
    }
}

// Copies of K/V tiles into LDS stages.  A tile is TILE_BYTES / 1024 instructions of 1 KiB, PIECES of
// them per wave, each lane fetching the 16-byte chunk that belongs at its (swizzled) LDS position; rows past the
// tile's valid ones arrive as zeros (they are the descriptor's size; a tile past the end of the
// key-tile list has none: zeros, no memory traffic).  The copy is issued from
// inline assembly on purpose: the compiler makes every later LDS read wait for all copies it
// knows of, also those into another stage, which would serialise the pipeline.  The waits are
// explicit instead (vmcnt before the barrier that publishes a stage).  Descriptor and LDS address
// are built from wave-uniform values on the scalar ALU; the compiler does not look into the
// assembly for hazards, so the statement carries its own wait states: one is what a scalar write
// of M0 needs, five would cover a descriptor word written by a vector instruction.
__device__ __forceinline__ void lds_copy_16(const u32x4& rsrc, uint32_t lds_addr, int voffset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds_addr), "v"(voffset), "s"(rsrc)
                 : "memory");                       // M0 has no other user in this file
}
// The same in two parts, for the loop: the LDS address goes into M0 a step before the copy that uses it, and
// the descriptor was built in the turn before, so that neither needs wait states (four of them cost a lone wave 20 cycles a copy).
// That holds as long as no scalar register is spilled: build.py refuses a build in which one is.
__device__ __forceinline__ void copy_to(uint32_t lds_addr) { asm volatile("s_mov_b32 m0, %0" :: "s"(lds_addr) : "memory"); }
__device__ __forceinline__ void copy_16(const u32x4& rsrc, int voffset) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen lds" :: "v"(voffset), "s"(rsrc) : "memory");
}
// Keeps a wave-uniform value in scalar registers (left to itself the compiler does the descriptor arithmetic on the
// vector ALU, with a 16-cycle multiplication per word).
__device__ __forceinline__ void scalar(uint32_t& x) { x = __builtin_amdgcn_readfirstlane(x); asm volatile("" : "+s"(x)); }
__device__ __forceinline__ void scalar(int& x) { x = __builtin_amdgcn_readfirstlane(x); asm volatile("" : "+s"(x)); }

// Byte offset of a K/V row, as two words.
struct RowOffset { uint32_t lo, hi; };
__device__ __forceinline__ RowOffset row_offset(const int row, const uint32_t row_bytes) {   // (row counts fit 31 bits)
    RowOffset r;
    const int row_s = __builtin_amdgcn_readfirstlane(row);
    asm volatile("s_mul_i32 %0, %1, %2" : "=s"(r.lo) : "s"(row_s), "s"(row_bytes));
    asm volatile("s_mul_hi_u32 %0, %1, %2" : "=s"(r.hi) : "s"(row_s), "s"(row_bytes));
    return r;
}
// Descriptor of a tile of `rows` valid rows at offset `off` of K or V (rows 0: empty), in two parts.
__device__ __forceinline__ void desc_base(u32x4& rs, const void* src, const RowOffset off) {
    const uint64_t s = reinterpret_cast<uint64_t>(src);
    uint32_t lo, hi;
    asm volatile("s_add_u32 %0, %2, %4\n\ts_addc_u32 %1, %3, %5\n\ts_and_b32 %1, %1, 0xffff"       // stride 0: raw buffer
                 : "=&s"(lo), "=&s"(hi) : "s"(off.lo), "s"(off.hi), "s"(static_cast<uint32_t>(s)), "s"(static_cast<uint32_t>(s >> 32)) : "scc");
    rs[0] = lo; rs[1] = hi; rs[3] = 0x00020000u;
}
__device__ __forceinline__ void desc_size(u32x4& rs, const uint32_t rows, const uint32_t row_bytes) {
    const uint32_t rows_s = __builtin_amdgcn_readfirstlane(rows);
    uint32_t size;
    asm volatile("s_mul_i32 %0, %1, %2" : "=s"(size) : "s"(rows_s), "s"(row_bytes));
    rs[2] = size;
}
__device__ __forceinline__ u32x4 tile_desc(const void* src, const RowOffset off, const uint32_t rows, const uint32_t row_bytes) {
    u32x4 rs;
    desc_base(rs, src, off);
    desc_size(rs, rows, row_bytes);
    return rs;
}
// this wave's piece Q (0 .. PIECES - 1) of a tile into the stage at byte offset DST
#define PK_COPY_PIECE(RS, DST, Q) lds_copy_16(RS, lds_wave + (DST) + ((Q) / PPS) * SLAB + ((Q) % PPS) * 1024, off.g[Q])
#define PK_COPY_TILE(RS, DST)                                                                \
    { _Pragma("unroll") for (int q = 0; q < PIECES; ++q) PK_COPY_PIECE(RS, DST, q); }
// What the loop needs of a list entry: how many keys there are to copy (none for an entry past the list) and, in bit 8, whether this
// wave has to mask the tile.  Codes of the list: 0 skip, 1 masked, 2 unmasked.
__device__ __forceinline__ int entry_info(const WorkUnit& u, const int ks, const int info, const int index) {
    const int keys = index < u.n_kv ? min(info & 0xFF, u.k_end - ks) : 0;
    const bool masked = ((info >> (8 + 2 * u.rows)) & 3) != 2 || ks + BN > u.full;
    return keys | (masked ? 0x100 : 0);
}

// ---------------------------------------------------------------------------------------------
// Five stages of LDS per workgroup, three for K and two for V.
// Softmax state of a query row.  The MFMAs work on Q and K as they are in memory, so a raw score is
// the exact sum of bf16 products in fp32; one fused multiply-add per score turns it into an exponent
// of two relative to the row's reference: x = sc * s - m_ref, sc = scale * log2 e.  (Folding sc
// into Q instead would save that instruction but costs another rounding of Q to bf16: 2^-9
// relative per element, which for scores of a few units' spread is an error of 0.03 .. 0.04 in
// the output, measured.)
//   m_ref   reference that the exponentials are taken against, in the exp2 domain.  It is set kSlack
//           above the row maximum it was taken from and only has to stay within a few dozen octaves
//           of the running one (bf16 and fp32 share their exponent range, so a probability of 2^-12
//           is as exact as one of 1), so it moves rarely ("lazy" rescaling).  kUnset: no key seen
//           yet, or a far reference (every visible score then asks for the slow path); kNoRow: no query
//           in this lane (every probability is 0);
//   far     a reference of 2^24 octaves or more (kNear) is a score instead, the row's maximum when it was taken,
//           and the exponents are formed in two steps, (s - far) * sc - kSlack: the rounding of m_ref is
//           32 octaves at 2^30, and from 2^31 on it would leave rows without a probability or with infinite
//           ones.  0: m_ref is the reference;
//   lsum[0] the row sum.
// Fast path of a half tile (8 scores per lane and column block): p = exp2(x), pairs rounded to bf16, no maximum, no
// sum.  The sum of a row is left to the matrix pipe: one MFMA per half tile and column block whose A operand is all
// ones.  It sums the ROUNDED probabilities, the numbers that go into P.V: a
// probability is taken against a reference that may lie far from the row maximum, so even a
// dominant one is not a round number, and its rounding error (2^-9 relative) has to cancel between
// numerator and denominator.  (With the unrounded values in the sum a row that one key dominates is
// off by 1.4e-2, with the rounded ones by 5e-3, measured.)  A column of the MFMAs is one query, so a probability that is
// not a number (a NaN or an infinity in Q or K) reaches the row that sees it and no other.
// Whether the reference is still good shows in the exponent bits of the packed pairs: if any
// probability is 2 or more (bit 14 of a bf16) the whole wave redoes the half tile on the slow path below,
// which finds the maximum, moves the reference and rescales what has been accumulated.  Scores that
// are still in the making (the other half tile's) are raw and meet the new reference when their
// turn comes.
struct HalfSoftmax {
    uint32_t any;                                  // all packed pairs or'ed together
    uint64_t slow;                                 // lanes that ask for the slow path
    uint32_t pw[4 * NC];                           // pairs of column block c: 4 c .. 4 c + 3
};
constexpr float kSlack = 12.f;                     // a fresh reference lies this far above the row maximum
constexpr float kRaiseBy = 8.f;                    // a set reference is only raised by more than this
constexpr float kNear = 16777216.f;                // below it fp32 rounds a reference by at most half an octave
constexpr float kUnset = -__FLT_MAX__, kNoRow = 1e30f;   // (kUnset lies below every scaled score that fp32 can hold)
constexpr uint32_t kTooLarge = 0x40004000u;        // a bf16 of 2 or more in either half

// max without the canonicalising self-maximum that fmaxf() costs per operand (scores are never NaN;
// -inf is ordinary here).  Not volatile: the compiler schedules these like any arithmetic.
__device__ __forceinline__ float max3f(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ float max2f(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The fast path of a half tile is dealt over the SLOTS MFMAs of a part, what stands behind MFMA `slot` here: an MFMA keeps
// the matrix pipe for 16 cycles, and a wave that has the next one ready stands there until it is free, so that what follows
// a run of MFMAs overlaps with the last of them only.  Of the vector ALU an MFMA takes 8 cycles, an exponential 8 and anything else
// 4, and a lone wave issues one instruction in 8.  Cycles for an MFMA and what stands behind it, one wave / two waves on a SIMD: alone 16.2 /
// 16.1, one multiply-add 16.3 / 16.1, an exponential 16.7 / 16.3, multiply-add and exponential of the same score 24.3 / 21.1, the exponential of
// one score and the multiply-add of the next 20.9 / 20.5; with a conversion behind every other MFMA 26.3 / 23.3 in the first order, 22.5 /
// 22.2 in the second.  So the exponential of a score stands a slot behind its multiply-add, and in front of the next one's, and the
// combination of the packed pairs a slot behind the conversion (one order / the other: 64 ragged prompts 383.0 / 377.2 us, 32 chunks of a 70B-shaped layer
// 10.58 / 10.49 ms, 8 x 2048 with head dimension 64 163.2 / 162.2 us, other shapes equal).
// The scores are through SPARE slots before the end and a pair is converted two slots behind its exponentials: neither
// the conversion nor the branch at the end waits for results.  Score e of a
// lane is element e & 3 of key block (e >> 2) & 1 of column block e >> 3.
typedef floatx4 Scores[NC][2];
struct Pending { float x[8]; };                    // exponents, then exponentials that are not packed yet
template <int SLOTS, int SPARE>
__device__ __forceinline__ void softmax_slot(const int slot, const Scores& s, const float sc, const float (&m_ref)[NC], Pending& p, HalfSoftmax& h) {
    constexpr int SCORES = 8 * NC;
    static_assert(SPARE == 0 || (SCORES - 1) * (SLOTS - SPARE) / SCORES + 4 < SLOTS, "every pair is packed and combined before the check behind the last slot");
    auto last = [](int at) { return at < SLOTS ? at : SLOTS; };
    auto begin = [](int e) { return e * (SLOTS - SPARE) / SCORES; };
#pragma unroll
    for (int e = 0; e < SCORES; ++e)
        if (last(begin(e) + 1) == slot) asm volatile("v_exp_f32 %0, %0" : "+v"(p.x[e & 7]));
#pragma unroll
    for (int k = 0; k < SCORES / 2; ++k) {
        if (last(begin(2 * k + 1) + 3) == slot)
            asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(h.pw[k]) : "v"(p.x[(2 * k) & 7]), "v"(p.x[(2 * k + 1) & 7]));
        if (last(begin(2 * k + 1) + 4) != slot) continue;
        if (k == 2) asm volatile("v_or3_b32 %0, %1, %2, %3" : "=v"(h.any) : "v"(h.pw[0]), "v"(h.pw[1]), "v"(h.pw[2]));
        else if (k > 2 && k % 2 == 0) asm volatile("v_or3_b32 %0, %0, %1, %2" : "+v"(h.any) : "v"(h.pw[k - 1]), "v"(h.pw[k]));
        else if (k == SCORES / 2 - 1) asm volatile("v_or_b32 %0, %0, %1" : "+v"(h.any) : "v"(h.pw[k]));
    }
#pragma unroll
    for (int e = 0; e < SCORES; ++e)
        if (begin(e) == slot)
            asm volatile("v_fma_f32 %0, %1, %2, -%3" : "=v"(p.x[e & 7]) : "v"(s[e >> 3][(e >> 2) & 1][e & 3]), "s"(sc), "v"(m_ref[e >> 3]));
    if (slot == (SPARE > 0 ? SLOTS - 1 : SLOTS)) {
        h.slow = __builtin_amdgcn_ballot_w64((h.any & kTooLarge) != 0);
        asm volatile("" : "+s"(h.slow));
    }
}

__device__ __forceinline__ float row_max(const floatx4 (&s)[2]) {   // the four lanes of a row agree through the swaps
    float mx = max3f(max3f(max3f(max2f(s[0][0], s[0][1]), s[0][2], s[0][3]), s[1][0], s[1][1]), s[1][2], s[1][3]);
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    mx = max2f(__uint_as_float(p[0]), __uint_as_float(p[1]));
    const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return max2f(__uint_as_float(q[0]), __uint_as_float(q[1]));
}
// A wave's first half tile: nothing has been accumulated, so the rows that see a key here take their
// reference before the exponentials (on the slow path they would be computed twice and the 64
// accumulators, all zero, rescaled: 0.4 us of vector work per query tile).  Far references are left to the slow path.
__device__ __forceinline__ void first_reference(const floatx4 (&s)[2], const float sc, float& m_ref) {
    const float fresh = __builtin_fmaf(row_max(s), sc, kSlack);
    if (__builtin_fabsf(fresh) < kNear) m_ref = max2f(m_ref, fresh);
}

// Slow path of a half tile (wave-uniform, rare): s holds the raw scores.  First the scalars: the
// row maximum (both lanes of a row agree through the swap), the new reference for the rows that
// need one, the factor alpha for what has been accumulated so far (0 for a row's first keys,
// when there is nothing).  The caller then recomputes the probabilities and rescales, each in a
// branch of its own that holds nothing but updates in place: written as one block, the paths join
// with the 64 accumulators in fresh registers, more than the kernel has.
// On this path a reference is far * sc + offset_of(m_ref, far), whichever of the two kinds it is.
__device__ __forceinline__ float offset_of(const float m_ref, const float far) { return far == 0.f ? m_ref : kSlack; }
__device__ __forceinline__ void softmax_slow_scalars(const floatx4 (&s)[2], const float sc, float& m_ref, float& far, float& alpha) {
    const float mx = row_max(s);                   // -inf for a row without a visible key here
    const float far0 = far, offset0 = offset_of(m_ref, far);
    if (__builtin_fmaf(mx - far, sc, -offset0) > kRaiseBy - kSlack) {
        const float fresh = __builtin_fmaf(mx, sc, kSlack);
        const bool near = __builtin_fabsf(fresh) < kNear;
        m_ref = near ? fresh : kUnset;
        far = near ? 0.f : mx;
    }
    alpha = __builtin_amdgcn_exp2f(__builtin_fmaf(far0 - far, sc, offset0 - offset_of(m_ref, far)));
}
__device__ __forceinline__ void softmax_redo(const floatx4 (&s)[2], uint32_t* pw, const float sc, const float m_ref, const float far) {
    const float offset = offset_of(m_ref, far);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float s0 = s[k >> 1][2 * (k & 1)], s1 = s[k >> 1][2 * (k & 1) + 1];
        pw[k] = pack_bf16x2(__builtin_amdgcn_exp2f(__builtin_fmaf(s0 - far, sc, -offset)),
                            __builtin_amdgcn_exp2f(__builtin_fmaf(s1 - far, sc, -offset)));
    }
}
// (The statements around the products keep them in place: the compiler would otherwise put the rescaled accumulators into fresh
// registers, more than there are.)
__device__ __forceinline__ void rescale(floatx4& x, const float alpha) {
    asm volatile("" : "+v"(x));
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] *= alpha;
    asm volatile("" : "+v"(x));
}
#define PK_SOFTMAX_CHECK(S, H)                                                                 \
    if (H.slow != 0) {                                                                         \
        float alpha[NC];                                                                       \
        PK_MFMA_RESULTS()                                                                      \
        _Pragma("unroll") for (int c = 0; c < NC; ++c) softmax_slow_scalars(S[c], sc, m_ref[c], far[c], alpha[c]); \
        _Pragma("unroll") for (int c = 0; c < NC; ++c) softmax_redo(S[c], H.pw + 4 * c, sc, m_ref[c], far[c]); \
        _Pragma("unroll") for (int c = 0; c < NC; ++c) {                                       \
            rescale(lsum[c], alpha[c]);                                                        \
            _Pragma("unroll") for (int t = 0; t < OPS; ++t) rescale(o[c][t], alpha[c]);        \
        }                                                                                      \
    }

// -inf for the keys of half `half` of a tile that a query row may not see.  A key tile lies inside the
// keys of one request, so a row either sees it from its first key on (up to its causal limit) or, being
// another request's, not at all: `visible` counts the tile's keys, from the first, that it sees.
__device__ __forceinline__ void mask_half(Scores& s, int half, const int (&visible)[2], int g) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int left = visible[c] - 4 * g - 32 * half;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (left <= 16 * k + j) s[c][k][j] = -INFINITY;
            asm volatile("" : "+v"(s[c][k]));   // ties the selects to this place, behind the caller's branch
        }
    }
}

// K operand x (0 .. OPS - 1) of a half tile: rows of key block x & 1, contraction step x / 2 (the two chains of
// scores take turns)
__device__ __forceinline__ bf16x8 k_operand(const unsigned char* const (&kp)[2], int half, int x) {
    const int s = x >> 1;
    return *reinterpret_cast<const bf16x8*>(kp[s & 1] + (s >> 1) * SLAB + (half * 32 + (x & 1) * 16) * SLAB_ROWB);
}
// Order of a part's 2 * OPS steps, one LDS operand and NC MFMAs each: of the scores (operand K) and of P.V (operand V).  Part A
// starts with four K operands, which can be read before the barrier that publishes the V tile; otherwise the two kinds
// take turns.
constexpr int NM = 2 * OPS;
constexpr int SPARE = D == 128 ? 2 * NC : 4;       // slots of a part behind its last score (at least four: softmax_slot)
constexpr bool op_is_v(int part, int m) {
    return part == 0 ? m >= 4 && (m >= NM - 4 || (m - 4) % 2 == 0) : m % 2 == 1;
}
constexpr int op_index(int part, int m) {
    int x = 0;
    for (int i = 0; i < m; ++i) x += op_is_v(part, i) == op_is_v(part, m);
    return x;
}
// piece of PK_ADVANCE behind MFMA c of step m: one each, or one in two, of the last 4 NC MFMAs
constexpr int advance_at(int m, int c) {
    const int q = (m - (NM - 4)) * NC + c;
    return q < 0 || q % (NC / 2) != 0 ? -1 : q / (NC / 2);
}
// Operand of step m of part `part` (0: A, 1: B; m >= NM: of the part that follows), or its piece PIECE of two: V operands
// take two reads, K operands one.  kp: this lane's two K addresses in the stage that is read; by the time the next part
// A's operands are read they are those of the next stage.
template <int PART, int M, int PIECE>
__device__ __forceinline__ void read_operand(bf16x8& op, bf16x4& half, const unsigned char* const (&kp)[2], const unsigned char* v_cur,
                                             const LaneOffsets& off) {
    constexpr int part = M < NM ? PART : 1 - PART, m = M < NM ? M : M - NM, x = op_index(part, m);
    if constexpr (!op_is_v(part, m)) { if constexpr (PIECE == 0) op = k_operand(kp, part, x); }
    else if constexpr (PIECE == 0) half = v_half_operand(v_cur, off, part, x, 0);
    else op = __builtin_shufflevector(half, v_half_operand(v_cur, off, part, x, 1), 0, 1, 2, 3, 4, 5, 6, 7);
}
#define PK_K_ADDRESSES(STAGE) _Pragma("unroll") for (int x = 0; x < 2; ++x) kp[x] = lds + (STAGE) + off.k[x];
// The MFMA, in place.  From the builtin the compiler makes the form with a destination of its own, and pays for it with copies
// of the accumulators wherever two paths join; and it moves the (side-effect free) arithmetic of the softmax and the
// MFMAs apart again, where the order of volatile statements stays.  What the compiler does not do for a statement is to wait for
// the result (a vector instruction may read it twelve wait states behind the last MFMA of the chain) and for operands that a
// vector instruction has written (two wait states).  In the loop other MFMAs are in between; elsewhere
// PK_MFMA_RESULTS() stands before the first reader and PK_MFMA_OPERANDS() before the MFMA.
__device__ __forceinline__ void mfma(floatx4& d, const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_out(floatx4& d, const bf16x8& a, const bf16x8& b) {     // (d: output accumulator)
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_first(floatx4& d, const bf16x8& a, const bf16x8& b) {   // d = a.b
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
#define PK_MFMA_OPERANDS() asm volatile("s_nop 1");
#define PK_MFMA_RESULTS() { asm volatile("s_nop 15"); __builtin_amdgcn_sched_barrier(0); }
// MFMA c of a step: scores of key block X & 1 / columns 16 X .. + 15 of P.V, and a row sum behind the last of each of the first NC
template <int X>
__device__ __forceinline__ void scores_mfma(const int c, Scores& s, const bf16x8& k, const bf16x8 (&qf)[NC][KS]) {
    if constexpr (X < 2) mfma_first(s[c][X & 1], k, qf[c][X >> 1]);
    else mfma(s[c][X & 1], k, qf[c][X >> 1]);
}
template <int X>
__device__ __forceinline__ void pv_mfma(const int c, floatx4 (&o)[NC][OPS], floatx4 (&lsum)[NC], const bf16x8& v, const bf16x8 (&p)[NC], const bf16x8& ones) {
    mfma_out(o[c][X], v, p[c]);
    if (X < NC && c == NC - 1) mfma_out(lsum[X < NC ? X : 0], ones, p[X < NC ? X : 0]);
}
// one step: NC MFMAs (MFMA, in terms of c), each with what stands behind it (SLOT, in terms of c)
#define PK_SLOT(C, MFMA, ...) if constexpr ((C) < NC) { constexpr int c = C; MFMA; __VA_ARGS__; __builtin_amdgcn_sched_barrier(0); }
#define PK_SLOTS(MFMA, ...) PK_SLOT(0, MFMA, __VA_ARGS__) PK_SLOT(1, MFMA, __VA_ARGS__)
// M: step of the part; DST: scores in the making; SRC: scores whose softmax is taken, into H; P: probabilities for P.V.  The ring
// holds operands M .. M + 2, and operand M + 3 replaces that of the step before.
#define PK_STEP_SLOT(PART, DST, SRC, H, P, EXTRA)                                             \
    softmax_slot<NM * NC, SPARE>(m * NC + c, SRC, sc, m_ref, pend, H);                         \
    if constexpr (c == NC - 1) { read_operand<PART, m + 4, 0>(ring[m & 3], ring_half, kp, lds + v_cur, off); read_operand<PART, m + 4, 1>(ring[m & 3], ring_half, kp, lds + v_cur, off); } \
    EXTRA
#define PK_STEP(PART, M, DST, SRC, H, P, EXTRA)                                               \
    {                                                                                          \
        constexpr int m = M, x = op_index(PART, m);                                            \
        if constexpr (op_is_v(PART, m)) {                                                      \
            PK_SLOTS((pv_mfma<x>(c, o, lsum, ring[m & 3], P, ones)), PK_STEP_SLOT(PART, DST, SRC, H, P, EXTRA)) \
        } else {                                                                               \
            PK_SLOTS((scores_mfma<x>(c, DST, ring[m & 3], qf)), PK_STEP_SLOT(PART, DST, SRC, H, P, EXTRA)) \
        }                                                                                      \
    }
#define PK_FOUR(PART, M, DST, SRC, H, P, EXTRA)                                               \
    PK_STEP(PART, (M), DST, SRC, H, P, EXTRA) PK_STEP(PART, (M) + 1, DST, SRC, H, P, EXTRA)    \
    PK_STEP(PART, (M) + 2, DST, SRC, H, P, EXTRA) PK_STEP(PART, (M) + 3, DST, SRC, H, P, EXTRA)
#if PK_D == 128
#define PK_PART(PART, DST, SRC, H, P, EXTRA)                                                  \
    {                                                                                          \
        Pending pend;                                                                          \
        PK_FOUR(PART, 0, DST, SRC, H, P, EXTRA) PK_FOUR(PART, 4, DST, SRC, H, P, EXTRA)        \
        PK_FOUR(PART, 8, DST, SRC, H, P, EXTRA) PK_FOUR(PART, 12, DST, SRC, H, P, EXTRA)       \
    }
#else
#define PK_PART(PART, DST, SRC, H, P, EXTRA)                                                  \
    {                                                                                          \
        Pending pend;                                                                          \
        PK_FOUR(PART, 0, DST, SRC, H, P, EXTRA) PK_FOUR(PART, 4, DST, SRC, H, P, EXTRA)        \
    }
#endif
// the OPS steps of one kind at the ends of a wave's tiles, step i
#define PK_OPS_STEP(I, ...) { constexpr int i = I; __VA_ARGS__; __builtin_amdgcn_sched_barrier(0); }
#define PK_OPS_FOUR(I, ...) PK_OPS_STEP(I, __VA_ARGS__) PK_OPS_STEP((I) + 1, __VA_ARGS__) PK_OPS_STEP((I) + 2, __VA_ARGS__) PK_OPS_STEP((I) + 3, __VA_ARGS__)
#if PK_D == 128
#define PK_OPS_STEPS(...) { PK_OPS_FOUR(0, __VA_ARGS__) PK_OPS_FOUR(4, __VA_ARGS__) }
#else
#define PK_OPS_STEPS(...) { PK_OPS_FOUR(0, __VA_ARGS__) }
#endif
#define PK_PACK_P(P, H)                                                                       \
    _Pragma("unroll") for (int c = 0; c < NC; ++c) {                                           \
        P[c] = __builtin_bit_cast(bf16x8, u32x4{H.pw[4 * c], H.pw[4 * c + 1], H.pw[4 * c + 2], H.pw[4 * c + 3]}); \
        asm volatile("" : "+v"(P[c]));                                                         \
    }

// `block`: the workgroup's number in the prefill launch order; `lds`: 5 * TILE_BYTES, 1 KiB aligned
// (K stages 0..2, V stages 3..4).
__device__ __forceinline__ void prefill_tile_body(const PrefillArgs& a, const int block, unsigned char* lds) {
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_ptr)lds));
    WorkUnit u;
    LaneOffsets off;
    bf16x8 qf[NC][KS];
    if (!setup(a, block, u, off, qf)) return;
    const int n_kv = u.n_kv;
    // The key-tile list, 64 entries at a time, one per lane: the loop takes entries out with v_readlane.  (A
    // scalar load shares its counter with the LDS reads and returns out of order: the wait for it drained the
    // operand ring, on the critical path of every tile.)  The next 64 are on their way.
    int list_s, list_i;
    int2 next_list = {0, 0};
    auto load_chunk = [&](int first) { return reinterpret_cast<const int2*>(u.kvt)[min(first + u.lane, n_kv - 1)]; };
    const int2 first_list = load_chunk(0);
    if (n_kv > 64) next_list = load_chunk(64);

    floatx4 o[NC][OPS], lsum[NC];
    float m_ref[NC], far[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        m_ref[c] = u.qrow[c] < 0 ? kNoRow : kUnset;   // rows without a query never ask for the slow path
        far[c] = 0.f;
        lsum[c] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < OPS; ++t) o[c][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
    asm volatile("" : "+v"(ones));                 // (not made again right before its MFMA)
    const float sc = a.scale * kLog2e;             // raw score -> exponent of two (the API admits only finite scale > 0)

    // this wave's 16 rows of a slab, as a scalar
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_base + u.wave * RPW * SLAB_ROWB);
    uint32_t row_bytes = u.row_bytes32;
    scalar(row_bytes);
#pragma unroll
    for (int x = 0; x < 3; ++x) u.info[x] = entry_info(u, u.ks[x], u.info[x], x);
    auto keys_of = [](int info) { return static_cast<uint32_t>(info & 0xFF); };
    // prologue: K(0), K(1), from the descriptor; the first turn copies K(2) and V(0)
    {
        const u32x4 rk0 = tile_desc(a.k, row_offset(u.ks[0], row_bytes), keys_of(u.info[0]), row_bytes);
        PK_COPY_TILE(rk0, 0)
        const u32x4 rk1 = tile_desc(a.k, row_offset(u.ks[1], row_bytes), keys_of(u.info[1]), row_bytes);
        PK_COPY_TILE(rk1, TILE_BYTES)
    }
    u32x4 rs_k = tile_desc(a.k, row_offset(u.ks[2], row_bytes), keys_of(u.info[2]), row_bytes);
    u32x4 rs_v = tile_desc(a.v, row_offset(u.ks[0], row_bytes), keys_of(u.info[0]), row_bytes);
    int es[4] = {u.ks[0], u.ks[0], u.ks[1], u.ks[2]}, ei[4] = {0, u.info[0], u.info[1], u.info[2]};   // list entries of tiles t .. t + 3
    int &cur_s = es[0], &cur_i = ei[0], &nxt_s = es[1], &nxt_i = ei[1];
#pragma unroll
    for (int x = 0; x < 4; ++x) { scalar(es[x]); scalar(ei[x]); }
#define PK_WAIT_AND_MEET() asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory")
    PK_WAIT_AND_MEET();
    list_s = first_list.x; list_i = entry_info(u, first_list.x, first_list.y, u.lane);
    clear_absent_rows(u, qf);

    bf16x8 ring[4];                                 // LDS operands of the next steps
    bf16x4 ring_half;                               // first half of one that takes two reads
    const unsigned char* kp[2];
    int k_cur = 0, k_next = TILE_BYTES, k_fill = 2 * TILE_BYTES;   // K stage read in this turn / in the next / filled now
    int v_cur = 4 * TILE_BYTES, v_fill = 3 * TILE_BYTES;
    copy_to(lds_wave + k_fill);
#define PK_PIECE_AT(Q) (((Q) / PPS) * SLAB + ((Q) % PPS) * 1024)
    // step I of a turn: copy I, and where copy I + 1 goes (copy 0: set at the end of the turn before)
#define PK_COPY_STEP(I) PK_COPY_ISSUE(I) PK_COPY_NEXT(I)
#define PK_COPY_ISSUE(I)                                                                      \
    if constexpr ((I) < PIECES) copy_16(rs_k, off.g[(I) < PIECES ? (I) : 0]);                  \
    else if constexpr ((I) < 2 * PIECES) copy_16(rs_v, off.g[(I) < 2 * PIECES ? (I) - PIECES : 0]);
#define PK_COPY_NEXT(I)                                                                       \
    if constexpr ((I) + 1 < PIECES) copy_to(lds_wave + k_fill + PK_PIECE_AT((I) + 1));         \
    else if constexpr ((I) + 1 < 2 * PIECES) copy_to(lds_wave + v_fill + PK_PIECE_AT((I) + 1 - PIECES));
    // The list entry of tile t + 4 and the next turn's descriptors, in eight pieces that stand behind the last MFMAs of a turn: done
    // behind the barrier they keep all waves of the workgroup from the matrix pipe at once.
#define PK_ADVANCE(I)                                                                         \
    if constexpr ((I) == 0) ek_s = __builtin_amdgcn_readlane(list_s, (t + 4) & 63);            \
    else if constexpr ((I) == 1) ek_i = __builtin_amdgcn_readlane(list_i, (t + 4) & 63);       \
    else if constexpr ((I) == 2) ek_off = row_offset(ek_s, row_bytes);                         \
    else if constexpr ((I) == 3) desc_base(rs_k, a.k, ek_off);                                 \
    else if constexpr ((I) == 4) desc_size(rs_k, keys_of(ek_i), row_bytes);          \
    else if constexpr ((I) == 5) ev_off = row_offset(es[2], row_bytes);                         \
    else if constexpr ((I) == 6) desc_base(rs_v, a.v, ev_off);                                 \
    else if constexpr ((I) == 7) desc_size(rs_v, keys_of(ei[2]), row_bytes);
#define PK_ADVANCE_ALL() PK_ADVANCE(0) PK_ADVANCE(1) PK_ADVANCE(2) PK_ADVANCE(3) PK_ADVANCE(4) PK_ADVANCE(5) PK_ADVANCE(6) PK_ADVANCE(7)
    // behind the last of 64 entries come the next 64, which were requested 64 turns ago (and nothing is on its way behind the barrier: taking
    // them waits for nothing)
#define PK_TURN_END()                                                                         \
    PK_WAIT_AND_MEET();                                                                        \
    if (((t + 4) & 63) == 63) {                                                                \
        list_s = next_list.x; list_i = entry_info(u, next_list.x, next_list.y, t + 5 + u.lane); \
        next_list = load_chunk(t + 5 + 64);                                                    \
    }                                                                                          \
    _Pragma("unroll") for (int x = 0; x < 3; ++x) { es[x] = es[x + 1]; ei[x] = ei[x + 1]; }   \
    es[3] = ek_s; ei[3] = ek_i;                                                                \
    _Pragma("unroll") for (int x = 0; x < 4; ++x) { scalar(es[x]); scalar(ei[x]); }            \
    { const int kc = k_cur; k_cur = k_next; k_next = k_fill; k_fill = kc; }                    \
    { const int vc = v_cur; v_cur = v_fill; v_fill = vc; }                                     \
    copy_to(lds_wave + k_fill);                                                                \
    ++t;
    // a turn in which this wave only takes part in the copies and the barrier
#define PK_SKIP_TURN()                                                                        \
    {                                                                                          \
        int ek_s, ek_i;                                                            \
        RowOffset ek_off, ev_off;                                                              \
        _Pragma("unroll") for (int q = 0; q < PIECES; ++q) { PK_COPY_PIECE(rs_k, k_fill, q); PK_COPY_PIECE(rs_v, v_fill, q); } \
        PK_ADVANCE_ALL()                                                                       \
        PK_TURN_END()                                                                          \
    }
    // mask of half `half` of a tile (the keys past its valid count are foreign)
    auto mask = [&](Scores& s, int half, int ks, int info) {
        int visible[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) visible[c] = u.lo[c] <= ks ? min(u.hi[c] - ks, info & 0xFF) : 0;
        mask_half(s, half, visible, u.g);
    };

    // Turn t = -1 .. n_kv - 1: P(t).V(t), the scores of tile t + 1 and the softmax of the halves (t, 1) and (t + 1, 0);
    // K(t + 3) and V(t + 1) are requested into the stages of K(t) and V(t - 1), one 1-KiB piece behind each of the
    // first 2 * PIECES steps, where their issue costs nothing.  The barrier at the end of a turn (after this
    // wave's copies have landed: only they matter, the compiler's own barrier would also wait for the LDS reads) says
    // that every wave is done with K(t + 1) and V(t) and that K(t + 3) and V(t + 1) are complete; K(t + 2), whose
    // first operands are read during the last MFMAs of the turn, was published a turn earlier.
    int t = -1;
    const bool any_tile = u.n_lead < u.n_active;
    const int first_turn = any_tile ? u.n_lead - 1 : -1;
    while (t < first_turn) PK_SKIP_TURN()
    if (any_tile) {
        Scores s0, s1;                              // scores of the first and of the second half of a tile
        HalfSoftmax h0, h1;
        bf16x8 p0[NC], p1[NC];
        bool masked = false;                        // tile t needs its mask
        {
            // first turn: the scores of this wave's first tile and the probabilities of its first half
            int ek_s, ek_i;
            RowOffset ek_off, ev_off;
            PK_K_ADDRESSES(k_cur)
#pragma unroll
            for (int x = 0; x < 4; ++x) ring[x] = k_operand(kp, 0, x);
            PK_OPS_STEPS(PK_SLOTS(scores_mfma<i>(c, s0, ring[i & 3], qf)) ring[i & 3] = k_operand(kp, (i + 4) / OPS, (i + 4) % OPS); PK_COPY_STEP(i))
            PK_MFMA_RESULTS()
            masked = (nxt_i & 0x100) != 0;
            if (masked) mask(s0, 0, nxt_s, nxt_i);
#pragma unroll
            for (int c = 0; c < NC; ++c) first_reference(s0[c], sc, m_ref[c]);
            Pending pend;
            PK_OPS_STEPS(PK_SLOTS(scores_mfma<i>(c, s1, ring[(OPS + i) & 3], qf), softmax_slot<OPS * NC, 0>(i * NC + c, s0, sc, m_ref, pend, h0))
                         if constexpr (i + 4 < OPS) ring[(OPS + i) & 3] = k_operand(kp, 1, i + 4))
            PK_ADVANCE_ALL()
            softmax_slot<OPS * NC, 0>(OPS * NC, s0, sc, m_ref, pend, h0);
            PK_SOFTMAX_CHECK(s0, h0)
            PK_PACK_P(p0, h0)
            PK_K_ADDRESSES(k_next)
#pragma unroll
            for (int x = 0; x < 4; ++x) ring[x] = k_operand(kp, 0, x);
            PK_TURN_END()
        }
        for (; t < u.n_active - 1;) {
            int ek_s, ek_i;
            RowOffset ek_off, ev_off;
            if (masked) mask(s1, 1, cur_s, cur_i);
            PK_PART(0, s0, s1, h1, p0, if constexpr (c == NC / 2) { PK_COPY_ISSUE(m) } if constexpr (c == NC - 1) { PK_COPY_NEXT(m) })
            PK_SOFTMAX_CHECK(s1, h1)
            PK_PACK_P(p1, h1)
            // (a tile that this wave could skip inside its active range is computed as a masked one)
            masked = (nxt_i & 0x100) != 0;
            if (masked) mask(s0, 0, nxt_s, nxt_i);
            PK_PART(1, s1, s0, h0, p1, if constexpr (m == NM - 5 && c == NC - 1) { PK_K_ADDRESSES(k_next) }
                    PK_ADVANCE(advance_at(m, c)))
            PK_SOFTMAX_CHECK(s0, h0)
            PK_PACK_P(p0, h0)
            PK_TURN_END()
        }
        {
            // Last turn: nothing but P.V and the probabilities of the last half, and no copies if it is the workgroup's last (nothing may
            // be on its way into LDS when that ends).  Of the rows of a causal tile every other wave's end in the first half of
            // their last key tile: the second half is left out then.
            if (t + 1 < n_kv) { _Pragma("unroll") for (int q = 0; q < PIECES; ++q) { PK_COPY_PIECE(rs_k, k_fill, q); PK_COPY_PIECE(rs_v, v_fill, q); } }
            const bool both = !masked || __builtin_amdgcn_ballot_w64((u.lo[0] <= cur_s && u.hi[0] - cur_s > 32) || (u.lo[1] <= cur_s && u.hi[1] - cur_s > 32)) != 0;
            if (masked) mask(s1, 1, cur_s, cur_i);
#pragma unroll
            for (int x = 0; x < 4; ++x) ring[x] = v_operand(lds + v_cur, off, 0, x);
            Pending pend;
            PK_OPS_STEPS(PK_SLOTS((pv_mfma<i>(c, o, lsum, ring[i & 3], p0, ones)), softmax_slot<OPS * NC, 0>(i * NC + c, s1, sc, m_ref, pend, h1))
                         ring[i & 3] = v_operand(lds + v_cur, off, (i + 4) / OPS, (i + 4) % OPS))
            softmax_slot<OPS * NC, 0>(OPS * NC, s1, sc, m_ref, pend, h1);
            if (both) {
                PK_SOFTMAX_CHECK(s1, h1)
                PK_PACK_P(p1, h1)
                PK_MFMA_OPERANDS()
                PK_OPS_STEPS(PK_SLOTS((pv_mfma<i>(c, o, lsum, ring[(OPS + i) & 3], p1, ones))) if constexpr (i + 4 < OPS) ring[(OPS + i) & 3] = v_operand(lds + v_cur, off, 1, i + 4))
            }
        }
    }
    PK_MFMA_RESULTS()
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(lsum[c]));   // (all four words of a sum are live until here)
    if (a.out_f32) store_output(a, u, o, lsum);
    else store_output_bf16(a, u, o, lsum);
    // The turns that are left for the other waves (the barrier at the end of the last one has nothing to wait for).
    if (any_tile && t < n_kv - 1) {
        int ek_s, ek_i;
        RowOffset ek_off, ev_off;
        PK_ADVANCE_ALL()
        PK_TURN_END()
    }
    while (t < n_kv - 1) PK_SKIP_TURN()
}

#undef PK_COPY_TILE
#undef PK_COPY_PIECE
#undef PK_COPY_STEP
#undef PK_PIECE_AT
#undef PK_SOFTMAX_CHECK
#undef PK_MFMA_RESULTS
#undef PK_MFMA_OPERANDS
#undef PK_STEP
#undef PK_STEP_SLOT
#undef PK_SLOT
#undef PK_SLOTS
#undef PK_FOUR
#undef PK_OPS_STEP
#undef PK_OPS_FOUR
#undef PK_COPY_ISSUE
#undef PK_COPY_NEXT
#undef PK_ADVANCE_ALL
#undef PK_PART
#undef PK_OPS_STEPS
#undef PK_PACK_P
#undef PK_WAIT_AND_MEET
#undef PK_TURN_END
#undef PK_SKIP_TURN
#undef PK_ADVANCE
#undef PK_K_ADDRESSES

}  // namespace PK_DNS
}  // namespace
}  // namespace pk
