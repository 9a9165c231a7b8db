// Packed prefill attention for launches of little work, bf16 MFMA, head dimension PK_D = 128 or 64 (Sec. 3.1).  Tables,
// arithmetic and copies are those of prefill_body.hip.h, with v_mfma_f32_32x32x16_bf16 and without a software pipeline over
// half tiles: no first and last turn, and half as many MFMAs for the same work, which is what counts for a wave that is alone on its
// SIMD, bound by the instructions it issues, one every five to six cycles.  Long launches are bound by power, which the 16x16x32 form uses
// less of; the schedule builder draws the line (light_launch in schedule.cpp, with both sides measured).
//   * a key tile is processed as two halves of 32 keys whose softmax steps are interleaved,
//     slice by slice, with the MFMAs of the neighbouring phase, and the LDS operand reads run
//     four MFMAs ahead in a ring of registers;
//   * copies are requested one tile ahead for V and two for K; one barrier per tile.

// Device code only: included by prefill_pipe.hip (the prefill launch) and by mixed_step.hip (the
// fused prefill + decode launch).  The includer defines PK_D (the head dimension) and PK_DNS (the namespace this
// instance goes into) first.  With PK_D = 64 a tile is 8 KiB instead of 16 and a
// half tile four MFMAs instead of eight, each followed by two softmax slices instead of one.
#include <cstdint>

#include "common.hip.h"
#include "kernels.h"

#if !defined(PK_D) || !defined(PK_DNS) || (PK_D != 128 && PK_D != 64)
#error "define PK_D (128 or 64) and PK_DNS before including prefill_few_body.hip.h"
#endif

namespace pk {
namespace {
namespace PK_DNS {

constexpr int BM = 128, BN = 64, D = PK_D;
constexpr int ROWB = D * 2;                        // bytes per K/V row in global memory
constexpr int TILE_BYTES = BN * ROWB;              // 16 KiB (8 KiB for D = 64)
constexpr int KS = D / 16, DB = D / 32;
constexpr int WAVES = 4;
constexpr int PIECES = TILE_BYTES / (1024 * WAVES);   // 1-KiB copy instructions per wave and tile
constexpr int RPW = BN / WAVES, PPS = RPW / 8;        // rows (and copies) of a slab that one wave fills
constexpr int WAVE_PART = TILE_BYTES / 4;          // bytes of a stage that take half of a wave's output

// A stage in LDS is one slab per 64 columns: 64 rows of 128 bytes (eight 16-byte chunks).  Whatever
// the head dimension, four K and four V addresses per lane then reach every operand with constant
// offsets, eight additions to the stage's address per key tile; with rows of 256 bytes it took eight of
// each and 24 additions, every sixth vector instruction of the loop.
constexpr int SLAB_ROWB = 128, SLAB = BN * SLAB_ROWB;

typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// Chunk position p of row `row` holds logical chunk p ^ swz(row).  Two 128-byte rows share a line of
// the 64 banks, so rows of the same parity need eight different values (K row reads of 16
// consecutive rows), and rows r and r + 2 must differ in bit 2 (the transpose reads take 64 bytes
// from each of four consecutive rows).
__device__ __forceinline__ int swz(int row) { const int x = (row >> 1) & 7; return ((x & 1) << 2) | (x >> 1); }

struct LaneOffsets {
    int k[4];           // K operand read: row n, logical chunk 2 (st & 3) + hlf of a slab
    int v1[2], v2[2];   // V transpose reads of column block b & 1 of a slab, rows +0..3 and +8..11
    int g[PIECES];      // global byte offsets of this lane's copy instructions
};

__device__ __forceinline__ bf16x8 v_operand(const unsigned char* vs, const LaneOffsets& lo, int kb, int t, int b) {
    const unsigned char* p = vs + (b >> 1) * SLAB + (32 * kb + 16 * t) * SLAB_ROWB;
    const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + lo.v1[b & 1]));
    const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + lo.v2[b & 1]));
    return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
}

// What a workgroup works on, and this lane's share of it.
struct WorkUnit {
    int head, kvh, n_kv, n_lead, n_active, wave, lane, n, hlf;   // this wave computes key tiles [n_lead, n_active)
    int rows;                          // which 32 of the tile's rows this wave has
    int ks[3], info[3];                // (first key row, info) of the tile's first three key tiles (the last one repeated)
    int qrow, lo, hi;                  // this lane's query row (-1: padding) and its key range [lo, hi)
    const int32_t* kvt;                // key-tile list of the query tile: (first key row, info) pairs
    int k_end, full;                   // keys from k_end on are not the tile's; up to `full` all of this wave's rows see them (row_shift < 2)
    int slot;                          // of this piece of a cut list (-1: the list is whole)
    int64_t record;                    // slot >= 0: where this wave's partial results go (PartialRecord)
    int64_t row_bytes;                 // bytes between consecutive K/V rows in global memory
    uint32_t row_bytes32;              // the same in 32 bits
};

// Decodes the workgroup id, loads the row metadata and the Q operand, derives the lane offsets.
// Returns false for grid padding and for query tiles without key tiles.
__device__ __forceinline__ bool setup(const PrefillArgs& a, const int block, WorkUnit& u, LaneOffsets& off, bf16x8 (&qf)[KS]) {
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
    u.slot = desc[15] - 1;
    const int tid = threadIdx.x;
    u.lane = tid & 63; u.n = u.lane & 31; u.hlf = u.lane >> 5;
    u.wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Wave w of every workgroup runs on SIMD w % 4, and the last rows of a causal tile see more key tiles than
    // the first: every other set of 256 workgroups (a set is one per compute unit) deals the rows in reverse,
    // so that the two waves of a SIMD get as much together as those of any other.
    const int part = u.wave & ((1 << a.row_shift) - 1), mate = u.wave >> a.row_shift;
    u.head = ((u.kvh * groups + group) << (2 - a.row_shift)) + mate;
    u.rows = (block >> 8) & 1 ? (1 << a.row_shift) - 1 - part : part;
    u.record = ((static_cast<int64_t>(u.slot) * a.Hkv + u.kvh) * groups + group) * WAVES + (mate << a.row_shift) + u.rows;
    u.n_active = u.n_kv - ((desc[3] >> (8 * u.rows)) & 0xFF);
    u.n_lead = min((desc[2] >> (8 * u.rows)) & 0xFF, u.n_active);
    prefill_tile_row(a, tile, desc[4], desc[5], desc[6], desc[7], u.rows * 32 + u.n, u.qrow, u.lo, u.hi);
    u.full = a.row_shift < 2 ? __builtin_amdgcn_readfirstlane(u.hi) : 0x7FFFFFFF;      // (the first row's; what one row sees, those behind it do)
    u.row_bytes = static_cast<int64_t>(a.Hkv) * ROWB;
    u.row_bytes32 = static_cast<uint32_t>(a.Hkv) * ROWB;

    const int fl = swz(u.n);
#pragma unroll
    for (int st = 0; st < 4; ++st) off.k[st] = u.n * SLAB_ROWB + (((2 * st + u.hlf) ^ fl) << 4);
    const int i16 = u.lane & 15, gl = (u.lane >> 4) & 1, r4 = i16 >> 2;
    const int rowl = 4 * u.hlf + r4, byte = (i16 & 1) * 8;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int c = 4 * b + 2 * gl + ((i16 & 3) >> 1);
        off.v1[b] = rowl * SLAB_ROWB + ((c ^ swz(rowl)) << 4) + byte;
        off.v2[b] = (rowl + 8) * SLAB_ROWB + ((c ^ swz(rowl + 8)) << 4) + byte;
    }
    const int r_in = u.lane >> 3, pos = u.lane & 7;    // a copy instruction takes 8 rows of 8 chunks
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int row = RPW * u.wave + 8 * (q % PPS) + r_in;
        off.g[q] = static_cast<int>(row * u.row_bytes + u.kvh * ROWB + (q / PPS) * SLAB_ROWB + ((pos ^ swz(row)) << 4));
    }
    // Q operand: lane (n, hlf) holds Q[row n][16s + 8hlf .. +8], as it is in memory: the MFMAs
    // deliver raw scores, exact products of the bf16 inputs summed in fp32.  Only requested here;
    // the first K/V copies follow at once, so that the two round trips to memory overlap.  Lanes without
    // a query read row 0 and are cleared once it is there (clear_absent_rows).
    const uint16_t* qp = static_cast<const uint16_t*>(a.q) +
                         (static_cast<int64_t>(u.qrow < 0 ? 0 : u.qrow) * a.Hq + u.head) * D + 8 * u.hlf;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qp + 16 * s));
    return true;
}

// Zeros for the lanes without a query: row 0, which they have read, is another request's and may hold anything.
__device__ __forceinline__ void clear_absent_rows(const WorkUnit& u, bf16x8 (&qf)[KS]) {
    if (__builtin_amdgcn_ballot_w64(u.qrow < 0) == 0) return;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        const u32x4 raw = __builtin_bit_cast(u32x4, qf[s]);
        qf[s] = __builtin_bit_cast(bf16x8, u.qrow < 0 ? u32x4{0u, 0u, 0u, 0u} : raw);
    }
}

// 1 / row sum (0 for a row without a visible key, NaN if either lane of the row holds one)
__device__ __forceinline__ float row_scale(const float l) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l), false, false);
    const float twice = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    return twice == 0.f ? 0.f : 2.f / twice;
}

// What a piece of a cut list leaves of the 32 rows and one head of a wave: its accumulators as they lie in the registers, and of every row the sum and the
// two words of its reference.  prefill_merge puts the pieces of a list together.
struct PartialRecord {
    floatx4 o[DB][4][64];
    floatx4 row[64];                               // row sum, m_ref, far
};
__device__ __forceinline__ __amdgpu_buffer_rsrc_t record_of(PartialRecord* p) {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, static_cast<int>(sizeof(PartialRecord)), 0x00020000);
}
__device__ __forceinline__ void store_partial(const PrefillArgs& a, const WorkUnit& u, const floatx16 (&o)[DB], const float l, const float m_ref, const float far) {
    if (__builtin_amdgcn_ballot_w64(u.qrow >= 0) == 0) return;
    const __amdgpu_buffer_rsrc_t rec = record_of(reinterpret_cast<PartialRecord*>(a.part) + u.record);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const floatx4 x = {o[b][4 * q4], o[b][4 * q4 + 1], o[b][4 * q4 + 2], o[b][4 * q4 + 3]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rec, 16 * u.lane, (4 * b + q4) * 1024, kWriteThrough);
        }
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, floatx4{l, m_ref, far, 0.f}), rec, 16 * u.lane, 4 * DB * 1024, kWriteThrough);
}

// o / l in fp32 to global memory; lane (n, hlf) owns columns 32b + 8q + 4hlf .. +3 of its query row.
__device__ __forceinline__ void store_output_f32(const PrefillArgs& a, const WorkUnit& u, const floatx16 (&o)[DB], const float l) {
    const float inv = row_scale(l);
    if (u.qrow < 0) return;
    float* out = static_cast<float*>(a.out) + (static_cast<int64_t>(u.qrow) * a.Hq + u.head) * D + 4 * u.hlf;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
            *reinterpret_cast<float4*>(out + 32 * b + 8 * q4) = make_float4(o[b][4 * q4] * inv, o[b][4 * q4 + 1] * inv, o[b][4 * q4 + 2] * inv, o[b][4 * q4 + 3] * inv);
}

// o / l through LDS, so that every row leaves as whole 16-byte pieces of ROWB bytes (four rows of 256
// bytes, or eight of 128, per store instruction) instead of 8- or 16-byte pieces of 32 different rows: bf16 rows at once, fp32 rows half by half.
// The wave uses two pieces of LDS of 16 rows each that belong to it alone (rows 0..15 in qa, rows
// 16..31 in qb); the 16-byte chunks of a row are XOR-swizzled with the row number, which keeps
// both sides off bank conflicts.
// Outputs of 2 MiB and more (PrefillArgs::through) are written through the L2.  What stays in it is written back when the launch is over, and beside decode work that streams its
// lines are evicted one at a time.  us, before / now: 15 x 30 rows with 32/8 heads 6.24 / 5.89, 20 x 24 with 64/8 8.21 / 7.36, 8 x 113 with 64/8 8.95 / 8.14, 4 x 436 with 32/8 and
// d = 64 20.1 / 19.1; the mixed step, 16 x 32 rows behind 100 with 32/8 beside 255 decode rows 216.8 / 202.7, 4 x 429 beside 276 64.6 / 58.9, 7 x 113 with 64/8 beside 3 12.1 / 10.7.  Smaller
// outputs wait longer for the memory than for the L2 (1 x 95 rows with 32/8, 0.8 MB: 11.6 / 11.9), and in fp32 go straight from the registers (LDS 0.5 us more).
template <bool F32>
__device__ __forceinline__ void store_output(const PrefillArgs& a, const WorkUnit& u, const floatx16 (&o)[DB],
                                             const float l, unsigned char* qa, unsigned char* qb) {
    constexpr int CPR = D / 8, RPI = 64 / CPR;     // 16-byte chunks per row; rows per store instruction
    const float inv = row_scale(l);
    const int rr = u.n & 15, chunk = u.lane & (CPR - 1);
    unsigned char* wrow = (u.n < 16 ? qa : qb) + rr * ROWB;
    int q_row[32 / RPI];
#pragma unroll
    for (int k = 0; k < 32 / RPI; ++k) q_row[k] = __shfl(u.qrow, RPI * k + u.lane / CPR, 64);
#pragma unroll
    for (int half = 0; half < (F32 ? 2 : 1); ++half) {
        constexpr int BLOCKS = F32 ? DB / 2 : DB;
#pragma unroll
        for (int b = 0; b < BLOCKS; ++b)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {       // columns 32 b + 8 q4 + 4 hlf .. + 3 (fp32: of this half)
                const floatx16& ob = o[half * BLOCKS + b];
                const float x0 = ob[4 * q4] * inv, x1 = ob[4 * q4 + 1] * inv, x2 = ob[4 * q4 + 2] * inv, x3 = ob[4 * q4 + 3] * inv;
                const int at = F32 ? 8 * b + 2 * q4 + u.hlf : 4 * b + q4;
                unsigned char* p = wrow + ((at ^ (rr & (CPR - 1))) << 4);
                if constexpr (F32) *reinterpret_cast<float4*>(p) = make_float4(x0, x1, x2, x3);
                else *reinterpret_cast<uint2*>(p + 8 * u.hlf) = make_uint2(pack_bf16x2(x0, x1), pack_bf16x2(x2, x3));
            }
        // all reads before the first store: one by one, each would wait for its own LDS round trips
        u32x4 v[32 / RPI];
#pragma unroll
        for (int k = 0; k < 32 / RPI; ++k) {
            const int row = RPI * k + u.lane / CPR, r2 = row & 15;
            v[k] = *reinterpret_cast<const u32x4*>((row < 16 ? qa : qb) + r2 * ROWB + ((chunk ^ (r2 & (CPR - 1))) << 4));
        }
        asm volatile("" ::: "memory");             // (the reads stay before the branches below)
        auto at = [&](const int k) {
            return static_cast<unsigned char*>(a.out) + (static_cast<int64_t>(q_row[k]) * a.Hq + u.head) * (F32 ? 2 * ROWB : ROWB) + half * ROWB + 16 * chunk;
        };
        if (F32 || a.through) {
#pragma unroll
            for (int k = 0; k < 32 / RPI; ++k)
                if (q_row[k] >= 0) write_through(at(k), v[k]);
        } else {
#pragma unroll
            for (int k = 0; k < 32 / RPI; ++k)
                if (q_row[k] >= 0) *reinterpret_cast<u32x4*>(at(k)) = v[k];
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
// Keeps a wave-uniform value in scalar registers (left to itself the compiler does the descriptor arithmetic on the
// vector ALU, with a 16-cycle multiplication per word).
__device__ __forceinline__ void scalar(uint32_t& x) { x = __builtin_amdgcn_readfirstlane(x); asm volatile("" : "+s"(x)); }
__device__ __forceinline__ void scalar(int& x) { x = __builtin_amdgcn_readfirstlane(x); asm volatile("" : "+s"(x)); }

// Byte offset of a K/V row, as two words.
struct RowOffset { uint32_t lo, hi; };
__device__ __forceinline__ RowOffset row_offset(const int row, const uint32_t row_bytes) {   // (row counts fit 31 bits)
    RowOffset r;
    const int row_s = __builtin_amdgcn_readfirstlane(row);
    asm("s_mul_i32 %0, %1, %2" : "=s"(r.lo) : "s"(row_s), "s"(row_bytes));
    asm("s_mul_hi_u32 %0, %1, %2" : "=s"(r.hi) : "s"(row_s), "s"(row_bytes));
    return r;
}
// descriptor of a tile of `rows` valid rows at offset `off` of K or V (rows 0: empty)
__device__ __forceinline__ u32x4 tile_desc(const void* src, const RowOffset off, const uint32_t rows, const uint32_t row_bytes) {
    const uint64_t s = reinterpret_cast<uint64_t>(src);
    uint32_t lo, hi, size;
    asm("s_add_u32 %0, %2, %4\n\ts_addc_u32 %1, %3, %5\n\ts_and_b32 %1, %1, 0xffff"       // stride 0: raw buffer
        : "=&s"(lo), "=&s"(hi) : "s"(off.lo), "s"(off.hi), "s"(static_cast<uint32_t>(s)), "s"(static_cast<uint32_t>(s >> 32)) : "scc");
    const uint32_t rows_s = __builtin_amdgcn_readfirstlane(rows);
    asm("s_mul_i32 %0, %1, %2" : "=s"(size) : "s"(rows_s), "s"(row_bytes));
    return u32x4{lo, hi, size, 0x00020000u};
}
// this wave's piece Q (0 .. PIECES - 1) of a tile into the stage at byte offset DST
#define PK_COPY_PIECE(RS, DST, Q) lds_copy_16(RS, lds_wave + (DST) + ((Q) / PPS) * SLAB + ((Q) % PPS) * 1024, off.g[Q])
#define PK_COPY_TILE(RS, DST)                                                                \
    { _Pragma("unroll") for (int q = 0; q < PIECES; ++q) PK_COPY_PIECE(RS, DST, q); }
#define PK_WAIT_ALL_COPIES() __builtin_amdgcn_s_waitcnt(0x0F70)      /* vmcnt(0) */
// What the loop needs of a list entry: how many keys there are to copy (none for an entry past the list) and, in bit 8, whether this
// wave has to mask the tile.  Codes of the list: 0 skip, 1 masked, 2 unmasked.
__device__ __forceinline__ int entry_info(const WorkUnit& u, const int ks, const int info, const int index) {
    const int keys = index < u.n_kv ? min(info & 0xFF, u.k_end - ks) : 0;
    const bool masked = ((info >> (8 + 2 * u.rows)) & 3) != 2 || ks + BN > u.full;
    return keys | (masked ? 0x100 : 0);
}

// ---------------------------------------------------------------------------------------------
// Two workgroups per CU, three with D = 64; five stages of LDS each, three for K and two for V.
// A key tile is handled as two halves of 32 keys, each with its own online-softmax step, so that
// within one wave the matrix pipe and the vector ALU overlap without state that crosses tiles:
//   phase 1   S0 = K(half 0) Q^T      with the requests for V(j+1), K(j+2)   (8 MFMAs + 2 * PIECES copies)
//   phase 2   S1 = K(half 1) Q^T      with the softmax of S0       (8 MFMAs + vector work)
//   phase 3   O += V(half 0)^T P0^T   with the softmax of S1       (8 MFMAs + vector work)
//   phase 4   O += V(half 1)^T P1^T                                (8 MFMAs)
//   barrier   this wave's copies have landed; every wave is done with the tile
// The LDS operand reads run four MFMAs ahead, in a ring of four operand registers that carries over
// the tile boundary (the first operands of tile j + 1 are read during the last MFMAs of tile j).
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
//   lsum[0] the row sum, over both halves of the wave; NaN once a score that this lane holds has given a
//           probability that is not a number (a NaN or an infinity in Q or K).
// Fast path of a half tile (16 scores per lane): p = exp2(x), pairs rounded to bf16, no maximum, no
// sum.  The sum of a row is left to the matrix pipe: one v_mfma_f32_16x16x32_bf16 per 16 keys
// whose A operand holds ones where they bring the sum of a query's P into register 0 of both
// lanes that carry it (row_sum_selector).  It sums the ROUNDED probabilities, the numbers that go into P.V: a
// probability is taken against a reference that may lie far from the row maximum, so even a
// dominant one is not a round number, and its rounding error (2^-9 relative) has to cancel between
// numerator and denominator.  (With the unrounded values in the sum a row that one key dominates is
// off by 1.4e-2, with the rounded ones by 5e-3, measured.)  A v_dot2_f32_bf16 per pair gives the same
// sum but costs as much as two and a half multiply-adds: in a loop of this kernel's mix (two
// waves per SIMD) 2.4 ns of 26.6 per 32x32x16 MFMA; the small MFMAs cost under 1.  On the whole kernel:
// 32 chunks of a 70B-shaped layer 11.85 -> 11.50 ms, 64 ragged prompts 436 -> 416 us, 8 long prompts
// with D = 64 604 -> 593 us.
// Whether the reference is still good shows in the exponent bits of the packed pairs: if any
// probability is 2 or more (bit 14 of a bf16) the whole wave redoes the half tile on the slow path below,
// which finds the maximum, moves the reference and rescales what has been accumulated.  Scores that
// are still in the making (the other half tile's) are raw and meet the new reference when their
// turn comes.
struct HalfSoftmax {
    uint32_t any;                                  // all packed pairs or'ed together
    uint32_t pw[8];
};
constexpr float kSlack = 12.f;                     // a fresh reference lies this far above the row maximum
constexpr float kRaiseBy = 8.f;                    // a set reference is only raised by more than this
constexpr float kNear = 16777216.f;                // below it fp32 rounds a reference by at most half an octave
constexpr float kUnset = -__FLT_MAX__, kNoRow = 1e30f;   // (kUnset lies below every scaled score that fp32 can hold)
constexpr uint32_t kTooLarge = 0x40004000u;        // a bf16 of 2 or more in either half

// A operand of the row-sum MFMA.  The B operand is P as the 32x32x16 MFMA takes it: lane l holds
// eight keys of query l & 31.  Seen as the operand of a 16x16x32 MFMA its lane group g = l / 16 is
// column l & 15, contraction block g; queries 0..15 sit in blocks 0 and 2, queries 16..31 in blocks
// 1 and 3.  Lane l receives rows 4 (l / 16) .. + 3 of its column: row 4 g takes the ones of the
// blocks with g's parity, the other rows are zero.
__device__ __forceinline__ bf16x8 row_sum_selector(int lane) {
    const int row = lane & 15, block = lane >> 4;
    const uint32_t w = (row & 3) == 0 && ((row >> 2) & 1) == (block & 1) ? 0x3F803F80u : 0u;
    return __builtin_bit_cast(bf16x8, u32x4{w, w, w, w});
}

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

// Slice C (0..7) of the fast path: pair C of the half tile, in two stages, so that the conversion
// never waits for its exponentials: stage A (fma, exp) right behind MFMA C, stage B (round, pack)
// behind MFMA C + 1 (1.4 % on the whole kernel; a third stage between fma and exp: nothing).
template <int C>
__device__ __forceinline__ floatx2 slice_a(const floatx16& s, const float sc, const float m_ref) {
    floatx2 pp;
    pp[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * C], sc, -m_ref));
    pp[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * C + 1], sc, -m_ref));
    return pp;
}
template <int C>
__device__ __forceinline__ void slice_b(const floatx2 pp, HalfSoftmax& h) {
    h.pw[C] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
    if constexpr (C == 0) h.any = h.pw[0];
    else if constexpr (C == 7) h.any |= h.pw[7];
    else if constexpr ((C & 1) == 0) h.any |= h.pw[C - 1] | h.pw[C];    // one v_or3_b32 every other slice
}

__device__ __forceinline__ float row_max(const floatx16& s) {      // both lanes of a row agree through the swap
    float mx = max3f(max3f(max3f(max2f(s[0], s[1]), s[2], s[3]), s[4], s[5]), s[6], s[7]);
    mx = max3f(max3f(max3f(max3f(mx, s[8], s[9]), s[10], s[11]), s[12], s[13]), s[14], s[15]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return max2f(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
}
// A wave's first half tile: nothing has been accumulated, so the rows that see a key here take their
// reference before the exponentials (on the slow path they would be computed twice and the 64
// accumulators, all zero, rescaled: 0.4 us of vector work per query tile).  Far references are left to the slow path.
__device__ __forceinline__ void first_reference(const floatx16& s, const float sc, float& m_ref) {
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
__device__ __forceinline__ void softmax_slow_scalars(const floatx16& s, const float sc, float& m_ref, float& far, float& alpha) {
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
__device__ __forceinline__ void softmax_redo(const floatx16& s, HalfSoftmax& h, const float sc, const float m_ref, const float far,
                                             const float alpha, floatx4& lsum) {
    const float offset = offset_of(m_ref, far);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        floatx2 pp;
        pp[0] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * q] - far, sc, -offset));
        pp[1] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[2 * q + 1] - far, sc, -offset));
        h.pw[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pp, bf16x2));
    }
    // With its reference in place a row's probabilities are below 2, unless one is a NaN.  None may reach the row-sum
    // MFMA, whose columns hold two queries and keep them apart by a factor of zero: the NaN goes to the lane's row sum
    // instead, and to no other row.
    uint32_t any = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) any |= h.pw[q];
    const bool bad = (any & kTooLarge) != 0;
    lsum[0] = bad ? __builtin_nanf("") : lsum[0] * alpha;
#pragma unroll
    for (int q = 0; q < 8; ++q) h.pw[q] = bad ? 0u : h.pw[q];
}
#define PK_SOFTMAX_CHECK(S, H)                                                                 \
    {                                                                                          \
        const bool slow = __builtin_amdgcn_ballot_w64((H.any & kTooLarge) != 0) != 0;          \
        float alpha = 1.f;                                                                     \
        /* the empty asm statements keep the compiler from computing the rare branches always */ \
        if (slow) { asm volatile(""); softmax_slow_scalars(S, sc, m_ref, far, alpha); }        \
        if (slow) { asm volatile(""); softmax_redo(S, H, sc, m_ref, far, alpha, lsum); }       \
        if (slow) {                                                                            \
            _Pragma("unroll") for (int b = 0; b < DB; ++b)                                     \
                _Pragma("unroll") for (int e = 0; e < 16; ++e) o[b][e] *= alpha;               \
        }                                                                                      \
    }

// The compiler is free to move the (side-effect free) softmax arithmetic and the MFMAs of a phase
// apart again.  Two empty volatile asm statements per slice tie them together: the first makes the
// slice's inputs depend on the point after MFMA i, the second makes the operand of MFMA i+1 depend
// on the point after the slice's results.
template <int C>
__device__ __forceinline__ void pin_slice_inputs(floatx16& acc, floatx16& s) {
    // (not after the first MFMA of a chain: tying its fresh result to the statement makes the
    // compiler copy the sixteen start values into it instead of naming them as the C operand)
    if constexpr (C == 0) asm volatile("" : "+v"(s));
    else asm volatile("" : "+v"(acc), "+v"(s));
}
template <int C>
__device__ __forceinline__ void pin_slice_outputs(bf16x8& next_operand, HalfSoftmax& h) {
    asm volatile("" : "+v"(next_operand), "+v"(h.pw[C]));
}

// -inf for the keys of half `half` of a tile that a query row may not see.  A key tile lies inside the
// keys of one request, so a row either sees it from its first key on (up to its causal limit) or, being
// another request's, not at all: `visible` counts the tile's keys, from the first, that it sees.
__device__ __forceinline__ void mask_half(floatx16& s, int half, int visible, int hlf) {
    const int left = visible - 4 * hlf - 32 * half;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        if (left <= 8 * (e >> 2) + (e & 3)) s[e] = -INFINITY;
        asm volatile("" : "+v"(s[e]));   // ties the selects to this place, behind the caller's branch
    }
}

// operand x (0..7) of a half tile: K rows of contraction step x; V^T block (t, b) = (x / 4, x % 4)
__device__ __forceinline__ bf16x8 k_operand(const unsigned char* const (&kp)[4], int half, int x) {
    return *reinterpret_cast<const bf16x8*>(kp[x & 3] + (x >> 2) * SLAB + half * 32 * SLAB_ROWB);
}
__device__ __forceinline__ bf16x8 v_operand_x(const unsigned char* vs, const LaneOffsets& lo, int half, int x) {
    return v_operand(vs, lo, half, x / DB, x % DB);
}
// Operand stream of a tile (KS operands per half tile; shown for D = 128): 0..7 K(half 0), 8..15
// K(half 1), 16..23 V(half 0), 24..31 V(half 1), 32..35 the first K operands of the next tile.
// MFMA k takes ring[k % 4] and then refills that slot with operand k + 4, so that every LDS read
// has four MFMAs (and their vector slices) to land.
template <int K>
__device__ __forceinline__ bf16x8 stream_operand(const unsigned char* const (&kp)[4], const unsigned char* v_cur,
                                                 const LaneOffsets& off) {
    if constexpr (K < 2 * KS) return k_operand(kp, K / KS, K % KS);
    else if constexpr (K < 4 * KS) return v_operand_x(v_cur, off, (K - 2 * KS) / KS, K % KS);
    else return k_operand(kp, 0, K - 4 * KS);      // (by then the addresses are those of the next tile)
}
// kp: this lane's four K addresses in the stage that is read; they move on to the next stage before
// phase 4, so that they are computed once per tile
#define PK_REFILL(K0) ring[i & 3] = stream_operand<(K0) + i + 4>(kp, lds + v_cur, off)
#define PK_K_ADDRESSES(STAGE) _Pragma("unroll") for (int x = 0; x < 4; ++x) kp[x] = lds + (STAGE) + off.k[x];
// the row sums of 16 keys, next to the first of the MFMAs that take the same P
#define PK_ROW_SUM(P) if constexpr (i % DB == 0) lsum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, P[i / DB], lsum, 0, 0, 0)
#define PK_SLICE(C, S, H, ACC, BODY)                                                          \
    {                                                                                          \
        constexpr int i = C;                                                                   \
        BODY;                                                                                  \
        pin_slice_inputs<C>(ACC, S);                                                           \
        if constexpr (C > 0) slice_b<(C > 0 ? C - 1 : 0)>(pend, H);                            \
        pend = slice_a<C>(S, sc, m_ref);                                                       \
        asm volatile("" : "+v"(pend));                                                         \
        pin_slice_outputs<(C > 0 ? C - 1 : 0)>(ring[(C + 1) & 3], H);                          \
    }
#if PK_D == 128
// eight MFMAs (BODY, with accumulator ACC) interleaved with the softmax of the scores S
#define PK_SLICES(S, H, ACC, BODY)                                                             \
    {                                                                                          \
    floatx2 pend;                                                                              \
    PK_SLICE(0, S, H, ACC, BODY) PK_SLICE(1, S, H, ACC, BODY) PK_SLICE(2, S, H, ACC, BODY)       \
    PK_SLICE(3, S, H, ACC, BODY) PK_SLICE(4, S, H, ACC, BODY) PK_SLICE(5, S, H, ACC, BODY)       \
    PK_SLICE(6, S, H, ACC, BODY) PK_SLICE(7, S, H, ACC, BODY)                                    \
    slice_b<7>(pend, H);                                                                       \
    }

#define PK_EIGHT(BODY)                                                                         \
    {                                                                                          \
        { constexpr int i = 0; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 1; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 2; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 3; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 4; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 5; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 6; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 7; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
    }
#else
// D = 64: four MFMAs per half tile, each followed by two of the eight softmax slices
#define PK_SLICE2(I, S, H, ACC, BODY)                                                          \
    {                                                                                          \
        constexpr int i = I;                                                                   \
        BODY;                                                                                  \
        pin_slice_inputs<I>(ACC, S);                                                           \
        if constexpr ((I) > 0) {                                                               \
            slice_b<((I) > 0 ? 2 * (I) - 2 : 0)>(pend, H);                                     \
            slice_b<((I) > 0 ? 2 * (I) - 1 : 1)>(pend2, H);                                    \
        }                                                                                      \
        pend = slice_a<2 * (I)>(S, sc, m_ref);                                                 \
        pend2 = slice_a<2 * (I) + 1>(S, sc, m_ref);                                            \
        asm volatile("" : "+v"(pend), "+v"(pend2));                                            \
        pin_slice_outputs<((I) > 0 ? 2 * (I) - 2 : 0)>(ring[((I) + 1) & 3], H);                \
        pin_slice_outputs<((I) > 0 ? 2 * (I) - 1 : 1)>(ring[((I) + 1) & 3], H);                \
    }
#define PK_SLICES(S, H, ACC, BODY)                                                             \
    {                                                                                          \
    floatx2 pend, pend2;                                                                       \
    PK_SLICE2(0, S, H, ACC, BODY) PK_SLICE2(1, S, H, ACC, BODY) PK_SLICE2(2, S, H, ACC, BODY)    \
    PK_SLICE2(3, S, H, ACC, BODY)                                                              \
    slice_b<6>(pend, H);                                                                       \
    slice_b<7>(pend2, H);                                                                      \
    }

#define PK_EIGHT(BODY)                                                                         \
    {                                                                                          \
        { constexpr int i = 0; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 1; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 2; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
        { constexpr int i = 3; BODY; __builtin_amdgcn_sched_barrier(0); }                      \
    }
#endif

// The rows of a tile whose list was cut: the partial results of its pieces, each weighted by its reference against the largest of them, in the order of
// their slots.  A workgroup has the 32 rows and one head of a wave of prefill_tile_body, wave b of it the columns 32 b .. + 31: `unit` counts (list, KV head,
// workgroup of the KV head, wave).  A reference is a score times sc and an offset (offset_of), so that those of far rows are subtracted before they are scaled.
// Bound by latency, two round trips to memory for every four pieces and 4 to 7 us with the launch.  A batch of four whole pieces has no checks between its sums and the last
// batch adds what there is: 1 x 64 rows behind 8000 with 8/8 heads 20.9 us, with a check for every piece 21.5, with zeros for the pieces that are not there 23.3.  (In the first launch instead, by the workgroup that finishes the last
// piece of a list: one workgroup then reads 68 KiB a piece, in a mixed step 3 x 90 rows behind some 9000 tokens with 4/1 heads 27.8 -> 43.3 us.)
__device__ __forceinline__ void prefill_merge(const PrefillArgs& a, const int unit) {
    constexpr int BATCH = 4;                       // pieces whose accumulators are requested together
    const int wid = unit & 3, x = unit >> 2, p = a.by_r(x), group = x - p * a.heads_per_kv, entry = a.by_hkv(p), kvh = p - entry * a.Hkv;
    const int32_t* e = a.merges + 4 * static_cast<int64_t>(entry);
    const int slot0 = e[0], pieces = e[1], q0 = e[2], n_rows = e[3];
    const int lane = threadIdx.x & 63, b = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)), n = lane & 31, hlf = lane >> 5;
    const int row = (wid & ((1 << a.row_shift) - 1)) * 32 + n;
    if (row - n >= n_rows) return;
    const int64_t stride = static_cast<int64_t>(a.Hkv) * a.heads_per_kv * WAVES;
    const PartialRecord* rec = reinterpret_cast<const PartialRecord*>(a.part) + ((static_cast<int64_t>(slot0) * a.Hkv + kvh) * a.heads_per_kv + group) * WAVES + wid;
    const float sc = a.scale * kLog2e;
    auto beyond = [&](const float m1, const float far1, const float m0, const float far0) {    // reference 1 minus reference 0, in octaves
        return __builtin_fmaf(far1 - far0, sc, offset_of(m1, far1) - offset_of(m0, far0));
    };
    float m = kUnset, far = 0.f;
    bool any = false;
    for (int s = 0; s < pieces; s += 2 * BATCH) {  // the reference farthest up
        floatx4 r[2 * BATCH];
#pragma unroll
        for (int y = 0; y < 2 * BATCH; ++y) r[y] = rec[min(s + y, pieces - 1) * stride].row[lane];
#pragma unroll
        for (int y = 0; y < 2 * BATCH; ++y)        // (a piece that a row sees nothing of has none; the last one repeated changes nothing)
            if (r[y][0] != 0.f && (!any || beyond(r[y][1], r[y][2], m, far) > 0.f)) { m = r[y][1]; far = r[y][2]; any = true; }
    }
    float l = 0.f;
    floatx4 o[4] = {};
    for (int s = 0; s < pieces; s += BATCH) {
        floatx4 r[BATCH], v[BATCH][4];
#pragma unroll
        for (int y = 0; y < BATCH; ++y) {
            const PartialRecord& t = rec[min(s + y, pieces - 1) * stride];
            r[y] = t.row[lane];
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) v[y][q4] = t.o[b][q4][lane];
        }
        asm volatile("" ::: "memory");             // (the reads stay before the branches below)
        auto add = [&](const int y) {
            const float w = r[y][0] != 0.f ? __builtin_amdgcn_exp2f(beyond(r[y][1], r[y][2], m, far)) : 0.f;
            l = __builtin_fmaf(w, r[y][0], l);
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                for (int c = 0; c < 4; ++c) o[q4][c] = __builtin_fmaf(w, v[y][q4][c], o[q4][c]);
        };
        if (s + BATCH <= pieces) {
#pragma unroll
            for (int y = 0; y < BATCH; ++y) add(y);
        } else {                                   // (not the last one repeated: a weight of zero would make NaNs of infinite values)
#pragma unroll
            for (int y = 0; y < BATCH - 1; ++y)
                if (s + y < pieces) add(y);
        }
    }
    const float inv = row_scale(l);
    if (row >= n_rows) return;
    const int head = ((kvh * a.heads_per_kv + group) << (2 - a.row_shift)) + (wid >> a.row_shift);
    const int64_t obase = (static_cast<int64_t>(q0 + row) * a.Hq + head) * D;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
        const int col = 32 * b + 8 * q4 + 4 * hlf;
        const floatx4 y = o[q4] * inv;
        if (a.out_f32) *reinterpret_cast<float4*>(static_cast<float*>(a.out) + obase + col) = make_float4(y[0], y[1], y[2], y[3]);
        else *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.out) + obase + col) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
    }
}

// `block`: the workgroup's number in the prefill launch order; `lds`: 5 * TILE_BYTES, 1 KiB aligned
// (K stages 0..2, V stages 3..4).
__device__ __forceinline__ void prefill_tile_body(const PrefillArgs& a, const int block, unsigned char* lds) {
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void_ptr)lds));
    WorkUnit u;
    LaneOffsets off;
    bf16x8 qf[KS];
    if (!setup(a, block, u, off, qf)) return;
    const int n_kv = u.n_kv;
    // The key-tile list, 64 entries at a time, one per lane: the loop takes the next entry out with v_readlane.  (A
    // scalar load shares its counter with the LDS reads and returns out of order: the wait for it drained the
    // operand ring, on the critical path of every tile.)
    int cur_s, cur_i, nxt_s, nxt_i;
    auto load_chunk = [&](int first, int& ks, int& info) {
        const int2 e = reinterpret_cast<const int2*>(u.kvt)[min(first + u.lane, n_kv - 1)];
        ks = e.x; info = e.y;
    };
    load_chunk(0, cur_s, cur_i);
    load_chunk(64, nxt_s, nxt_i);

    floatx16 o[DB];
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[b][e] = 0.f;
    float m_ref = u.qrow < 0 ? kNoRow : kUnset;    // rows without a query never ask for the slow path
    float far = 0.f;
    floatx4 lsum = {0.f, 0.f, 0.f, 0.f};
    const bf16x8 ones = row_sum_selector(u.lane);
    const floatx16 zero16 = {};
    const float sc = a.scale * kLog2e;             // raw score -> exponent of two (the API admits only finite scale > 0)

    // this wave's 16 rows of a slab, as a scalar
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_base + u.wave * RPW * SLAB_ROWB);
    // window of tile-list entries: e0 = tile j, e1 = tile j+1, e2 = tile j+2; what the loop copies in tile j is
    // K(j+2) and V(j+1)
#pragma unroll
    for (int x = 0; x < 3; ++x) u.info[x] = entry_info(u, u.ks[x], u.info[x], x);
    int e0s = u.ks[0], e0i = u.info[0], e1i = u.info[1], e1s = u.ks[1], e2s = u.ks[2], e2i = u.info[2];
    scalar(e0s); scalar(e0i); scalar(e1s); scalar(e1i); scalar(e2s); scalar(e2i);
    uint32_t row_bytes = u.row_bytes32;
    scalar(row_bytes);
    auto keys_of = [](int info) { return static_cast<uint32_t>(info & 0xFF); };
    // prologue: K(0), K(1), V(0), from the descriptor
    {
        const u32x4 rk0 = tile_desc(a.k, row_offset(e0s, row_bytes), keys_of(e0i), row_bytes);
        PK_COPY_TILE(rk0, 0)
        const u32x4 rk1 = tile_desc(a.k, row_offset(e1s, row_bytes), keys_of(e1i), row_bytes);
        PK_COPY_TILE(rk1, TILE_BYTES)
        const u32x4 rv0 = tile_desc(a.v, row_offset(e0s, row_bytes), keys_of(e0i), row_bytes);
        PK_COPY_TILE(rv0, 3 * TILE_BYTES)
    }
    RowOffset off2 = row_offset(e2s, row_bytes);             // of tile j+2
    u32x4 rs_k = tile_desc(a.k, off2, keys_of(e2i), row_bytes);
    u32x4 rs_v = tile_desc(a.v, row_offset(e1s, row_bytes), keys_of(e1i), row_bytes);
    PK_WAIT_ALL_COPIES();
    __syncthreads();
    cur_i = entry_info(u, cur_s, cur_i, u.lane);
    clear_absent_rows(u, qf);

    bf16x8 ring[4];                                 // LDS operands of the next four MFMAs
    const unsigned char* kp[4];
    PK_K_ADDRESSES(0)
#pragma unroll
    for (int x = 0; x < 4; ++x) ring[x] = k_operand(kp, 0, x);
    int k_cur = 0, k_next = TILE_BYTES, k_fill = 2 * TILE_BYTES;   // K stage read now / next / filled now
    int v_cur = 3 * TILE_BYTES, v_fill = 4 * TILE_BYTES;
    // Tile j: while S0 is computed, V(j+1) and K(j+2) are requested into the stages of V(j-1) and
    // K(j-1), one 1-KiB piece behind each of the first 2 * PIECES MFMAs, where their issue costs nothing.  The
    // barrier at the END of the tile (after this wave's copies have landed: only they matter, the
    // compiler's own barrier would also wait for the LDS reads) says that every wave is done with
    // tile j and that V(j+1) and K(j+2) are complete; K(j+1), whose first operands are read during
    // the last MFMAs of tile j, was published a tile earlier.
#define PK_COPY_STEP(I)                                                                       \
    if constexpr ((I) < PIECES) PK_COPY_PIECE(rs_k, k_fill, (I));                              \
    else if constexpr ((I) < 2 * PIECES) PK_COPY_PIECE(rs_v, v_fill, (I) - PIECES);
    // The next tile's list entry and descriptors, in four steps that stand between the last MFMAs of a tile: done
    // behind the barrier they keep all waves of the workgroup from the matrix pipe at once.
#define PK_ADVANCE(I)                                                                         \
    if constexpr ((I) == 0) {                                                                  \
        e3s = __builtin_amdgcn_readlane(cur_s, (j + 3) & 63); e3i = __builtin_amdgcn_readlane(cur_i, (j + 3) & 63); \
        rs_v = tile_desc(a.v, off2, keys_of(e2i), row_bytes);                    \
    } else if constexpr ((I) == 1) {                                                           \
        off2 = row_offset(e3s, row_bytes);                                                             \
    } else if constexpr ((I) == 2) {                                                           \
        rs_k = tile_desc(a.k, off2, keys_of(e3i), row_bytes);                    \
    }
    // entry j + 3 is the first of the next 64
#define PK_NEXT_CHUNK()                                                                       \
    if (((j + 3) & 63) == 0) {                                                                 \
        cur_s = nxt_s; cur_i = entry_info(u, nxt_s, nxt_i, j + 3 + u.lane);                    \
        load_chunk(j + 3 + 64, nxt_s, nxt_i);                                                  \
    }
#define PK_TILE_END()                                                                         \
    asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");                              \
    e0s = e1s; e0i = e1i; e1s = e2s; e1i = e2i; e2s = e3s; e2i = e3i;                          \
    scalar(e0s); scalar(e0i); scalar(e1s); scalar(e1i); scalar(e2s); scalar(e2i);              \
    { const int kc = k_cur; k_cur = k_next; k_next = k_fill; k_fill = kc; }                    \
    { const int vc = v_cur; v_cur = v_fill; v_fill = vc; }
#define PK_SKIP_TILE()                                                                        \
    {                                                                                          \
        int e3s, e3i;                                                                          \
        _Pragma("unroll") for (int q = 0; q < PIECES; ++q) { PK_COPY_PIECE(rs_k, k_fill, q); PK_COPY_PIECE(rs_v, v_fill, q); } \
        PK_NEXT_CHUNK()                                                                        \
        PK_ADVANCE(0) PK_ADVANCE(1) PK_ADVANCE(2)                                              \
        PK_TILE_END()                                                                          \
    }

    int j = 0;
    // leading tiles that this wave skips: it only takes part in the copies and in the barriers,
    // then picks up its first operands from the stage that is current by then
    for (; j < u.n_lead; ++j) {
        PK_SKIP_TILE()
    }
    if (u.n_lead > 0) {
        PK_K_ADDRESSES(k_cur)
#pragma unroll
        for (int x = 0; x < 4; ++x) ring[x] = k_operand(kp, 0, x);
    }
    for (; j < u.n_active; ++j) {
        // a tile that this wave could skip inside its active range is computed as a masked one
        const bool masked = (e0i & 0x100) != 0, special = masked || j == u.n_lead;
        // (keys past the tile's valid count are foreign)
        const int visible = u.lo <= e0s ? min(u.hi - e0s, e0i & 0xFF) : 0;
        int e3s, e3i;
        floatx16 s0, s1;
        PK_EIGHT(s0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i & 3], qf[i], i == 0 ? zero16 : s0, 0, 0, 0);
                 PK_REFILL(0); PK_COPY_STEP(i));
        HalfSoftmax h0, h1;
        if (special) {                              // (one branch in the common case)
            if (masked) mask_half(s0, 0, visible, u.hlf);
            if (j == u.n_lead) { asm volatile(""); first_reference(s0, sc, m_ref); }
        }
        PK_SLICES(s0, h0, s1, s1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i & 3], qf[i], i == 0 ? zero16 : s1, 0, 0, 0);
                  PK_REFILL(KS));
        PK_SOFTMAX_CHECK(s0, h0)
        bf16x8 p0[2], p1[2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
            p0[t] = __builtin_bit_cast(bf16x8, u32x4{h0.pw[4 * t], h0.pw[4 * t + 1], h0.pw[4 * t + 2], h0.pw[4 * t + 3]});
        if (masked) mask_half(s1, 1, visible, u.hlf);
        PK_SLICES(s1, h1, o[i % DB], o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i & 3], p0[i / DB], o[i % DB], 0, 0, 0);
                  PK_ROW_SUM(p0); PK_REFILL(2 * KS));
        PK_SOFTMAX_CHECK(s1, h1)
#pragma unroll
        for (int t = 0; t < 2; ++t)
            p1[t] = __builtin_bit_cast(bf16x8, u32x4{h1.pw[4 * t], h1.pw[4 * t + 1], h1.pw[4 * t + 2], h1.pw[4 * t + 3]});
        // phase 4; its last refills are the first operands of the next tile
        PK_NEXT_CHUNK()
        PK_K_ADDRESSES(k_next)
        PK_EIGHT(o[i % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[i & 3], p1[i / DB], o[i % DB], 0, 0, 0);
                 PK_ROW_SUM(p1); PK_REFILL(3 * KS); PK_ADVANCE(i));
        PK_TILE_END();
    }
    // trailing tiles that this wave skips: it only takes part in the copies and in the barriers
    for (; j < n_kv; ++j) {
        PK_SKIP_TILE()
    }
    // After the last barrier nobody fills a stage any more, and what is still being read for a tile after
    // the last is not used: quarters of a K and a V stage stage the waves' output.
    PK_WAIT_ALL_COPIES();                          // (none is outstanding here; kept as a guard)
    if (u.slot >= 0) store_partial(a, u, o, lsum[0], m_ref, far);
    else if (a.out_f32 && !a.through) store_output_f32(a, u, o, lsum[0]);
    else if (a.out_f32) store_output<true>(a, u, o, lsum[0], lds + k_next + u.wave * WAVE_PART, lds + v_cur + u.wave * WAVE_PART);
    else store_output<false>(a, u, o, lsum[0], lds + k_next + u.wave * WAVE_PART, lds + v_cur + u.wave * WAVE_PART);
}

#undef PK_COPY_TILE
#undef PK_COPY_PIECE
#undef PK_COPY_STEP
#undef PK_SOFTMAX_CHECK
#undef PK_ADVANCE
#undef PK_NEXT_CHUNK
#undef PK_SKIP_TILE
#undef PK_TILE_END
#undef PK_SLICE
#undef PK_SLICE2
#undef PK_SLICES
#undef PK_EIGHT
#undef PK_REFILL
#undef PK_ROW_SUM
#undef PK_K_ADDRESSES
#undef PK_WAIT_ALL_COPIES

}  // namespace PK_DNS
}  // namespace
}  // namespace pk
