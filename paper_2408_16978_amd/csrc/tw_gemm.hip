// Dense bf16 products of the token-wise chunked operations (Sec. 4.1, 5.4: the per-chunk QKV
// projection, the feed-forward block and the output projection of the loss are plain GEMMs over
// one chunk of tokens at a time) on v_mfma_f32_16x16x32_bf16: stages of 64 k in LDS, filled by direct
// global -> LDS copies two stages ahead, four waves (one per SIMD) per output tile of up to
// 256 x 256.
//
//   C[M,N] (+)= sum_k Aop[m,k] * Bop[n,k]          fp32 accumulation, C bf16 or fp32
//
// Every product of the library is of this form once each operand is read either as stored
// (row = row, k = column) or transposed (row = column, k = row).  Both are read in place: the copy
// engine fetches 16-byte pieces of the stored rows, a plain LDS read delivers the fragments of the
// first form and a transposing LDS read those of the second.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "mfma_tiles.h"
#include "tw_gemm.h"
#include "tw_plan.h"

namespace fpdt_tw {

using fpdt::bf16x8;
using fpdt::floatx4;
using fpdt::u32x4;

namespace {

// ---- realign ----------------------------------------------------------------------------
// The product kernel copies 16-byte pieces of its operands' rows.  An operand that does not offer that (a
// width that is not a multiple of 8, a base that is not 16-byte aligned), or that the product overwrites, is
// copied once: X [R, C] with its columns rounded up to 8, zero behind C, rows `pitch` elements apart.
__global__ __launch_bounds__(256) void tw_realign_kernel(const uint16_t* __restrict__ X, int64_t R, int64_t C, int64_t ld,
                                                         u32x4* __restrict__ out, int64_t pitch)
{
    const int64_t pieces = (C + 7) / 8, n = R * pieces;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t r = n >> 32 ? i / pieces : (unsigned)i / (unsigned)pieces, c = (i - r * pieces) * 8;
        u32x4 v;
        if (c + 8 <= C) {  // (16 bytes at any even address in one access)
            __builtin_memcpy(&v, X + r * ld + c, 16);
        } else {
            unsigned e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = c + j < C ? X[r * ld + c + j] : 0u;
            v = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        }
        out[r * (pitch / 8) + c / 8] = v;
    }
}

// ---- product ----------------------------------------------------------------------------
constexpr int NWAVE = 4, NTHREAD = NWAVE * 64;
constexpr unsigned PANEL = 8192;  // bytes of a panel: 64 rows of one operand x STAGE_K

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
// eight values rounded to nearest even, two per instruction
__device__ __forceinline__ u32x4 pack_bf16(floatx4 lo, floatx4 hi)
{
    const fpdt::floatx8 x = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(u32x4, __builtin_convertvector(x, bf16x8));
}
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((unsigned)b << 16); }

// Sum in fp32, stored as fp32 or bf16
template <bool ACC>
__device__ __forceinline__ float combine(float v, float old) { return ACC ? old + v : v; }
template <bool ACC>
__device__ __forceinline__ uint16_t combine(float v, uint16_t old) { return to_bf16(ACC ? from_bf16(old) + v : v); }

// One operand as stored: row r at p + r * ld, 16-byte aligned, ld a multiple of 8.  Form N: rows are the
// product's rows, columns its k.  Form T: rows are k, columns the product's rows.  `rows` counts the
// product's rows (form T: rounded up to 8, in bounds).
struct Operand {
    const uint16_t* p;
    int64_t ld;
    int rows;
};

// Per-lane source of one operand's copies and fragment reads.  A stage of an operand is PANEL bytes per 64
// rows, in eight copies of 1 KiB; wave w makes copies w and w + 4 of every panel.  Both forms read whole
// 128-byte lines: stages of half as many k, with 64 bytes of a row of form N, moved every line from L2
// twice (copies alone: 70 bytes per ns and compute unit against 140).
//   Form N: panel row r (128 bytes) holds its eight 16-byte pieces q at position q ^ (r / 2) % 8: the sixteen
//           lanes that a 16-byte read serves at a time (0-3, 12-15, 20-23 and 24-27 of 32, then the others)
//           lie in different 16-byte columns of 256 bytes.
//   Form T: two halves of 32 k; panel row k (128 bytes, 64 columns) holds its 32-byte quarter u at
//           u ^ (2 ((k / 2) % 2) + (k / 8) % 2): the eight k x 16 columns that half a wave's transposing read
//           covers lie in different 32-byte columns of 256 bytes.
__device__ __forceinline__ int piece_swizzle(int row) { return (row >> 1) & 7; }
template <bool T, int NP>
struct Side {
    uint64_t pos;           // scalar: the stage that is copied next
    uint64_t step;          // bytes from a stage to the next
    uint64_t half;          // form T: bytes from the rows of copy w to those of copy w + 4
    unsigned off[2][NP];    // this lane's piece of panel j, copies w and w + 4
    unsigned rd[T ? 4 : 2];  // LDS bytes within a stage.  T: of fragments 0, 4, .., of 1, 5, ..; N: of the two k-steps

    __device__ __forceinline__ void init(const Operand& x, int row0, int stage0, int w, int wave_frag0, int lane, unsigned lds0)
    {
        const uint64_t pitch = (uint64_t)x.ld * 2;
        const int limit = x.rows - row0;  // >= 1
        if constexpr (T) {
            step = STAGE_K * pitch;
            half = 32 * pitch;
            pos = (uint64_t)(uintptr_t)(x.p + row0) + (uint64_t)stage0 * step + (uint64_t)(8 * w) * pitch;
            const int k = lane >> 3, u = ((lane >> 1) & 3) ^ (2 * ((k >> 1) & 1) + (w & 1));
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int c = 64 * j + 16 * u + 8 * (lane & 1);
                off[0][j] = off[1][j] = (unsigned)k * (unsigned)pitch + 2u * (unsigned)(c < limit - 8 ? c : limit - 8);
            }
            // 16-lane group g supplies k rows 8 g + 0..3 (and + 4..7 with the second read), lane i of it row
            // i / 4, columns 4 (i % 4) .. + 3
            const int g = lane >> 4, e = (lane & 15) >> 2;
            const unsigned lane_part = 128u * (unsigned)(8 * g + e) + 8u * (unsigned)(lane & 3);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int f = wave_frag0 + q;
                rd[q] = lds0 + PANEL * (unsigned)(f >> 2) + 32u * (unsigned)((f & 3) ^ (2 * (e >> 1) + (g & 1))) + lane_part;
            }
        } else {
            step = STAGE_K * 2;
            half = 0;
            pos = (uint64_t)(uintptr_t)x.p + (uint64_t)row0 * pitch + (uint64_t)stage0 * step;
            const int r = lane >> 3, q = (lane & 7) ^ piece_swizzle(8 * w + r);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    // rows behind the operand are read as its last row: their products are not stored
                    const int mine = 64 * j + 32 * h + 8 * w + r < limit ? 64 * j + 32 * h + 8 * w + r : limit - 1;
                    off[h][j] = (unsigned)mine * (unsigned)pitch + 16u * (unsigned)q;
                }
            const int fr = lane & 15;
            rd[0] = lds0 + 128u * (unsigned)(16 * wave_frag0 + fr) + 16u * (unsigned)((lane >> 4) ^ piece_swizzle(fr));
            rd[1] = rd[0] ^ 64u;
        }
        pos = fpdt::uniform(pos);
    }
    // The copies of the last `k_left` < STAGE_K of k, with pos at their stage: what lies behind them is fetched
    // from where k is in range instead (and cleared by clear_tail).
    __device__ __forceinline__ void turn_to_tail(const Operand& x, int k_left, int w, int lane)
    {
        if constexpr (T) {
            const uint64_t pitch = (uint64_t)x.ld * 2;
            const int first0 = 8 * w < k_left ? 8 * w : k_left - 1, first1 = 8 * w + 32 < k_left ? 8 * w + 32 : k_left - 1;
            pos = fpdt::uniform(pos - (uint64_t)(8 * w - first0) * pitch);
            half = (uint64_t)(first1 - first0) * pitch;
            const int k = lane >> 3;
            const int back0 = k > k_left - 1 - first0 ? k - (k_left - 1 - first0) : 0, back1 = k > k_left - 1 - first1 ? k - (k_left - 1 - first1) : 0;
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                off[0][j] -= (unsigned)back0 * (unsigned)pitch;
                off[1][j] -= (unsigned)back1 * (unsigned)pitch;
            }
        } else {
            const int q = (lane & 7) ^ piece_swizzle(8 * w + (lane >> 3));
            const unsigned back = 8 * q < k_left ? 0u : 16u * (unsigned)q;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < NP; ++j) off[h][j] -= back;
        }
        step = 0;
    }
    // Zeros into this lane's pieces of a stage of which `k_left` < STAGE_K of k are in range (form N: rounded up to
    // 8); lds0: this wave's first piece of the operand in the slot
    __device__ __forceinline__ void clear_tail(int k_left, int w, int lane, unsigned lds0) const
    {
        typedef __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = T ? 32 * h + 8 * w + (lane >> 3) : 8 * ((lane & 7) ^ piece_swizzle(8 * w + (lane >> 3)));
            if (k >= k_left)
#pragma unroll
                for (int j = 0; j < NP; ++j) *(lds_u32x4_ptr)(uintptr_t)(lds0 + PANEL * (unsigned)j + 4096u * (unsigned)h + 16u * (unsigned)lane) = u32x4{0, 0, 0, 0};
        }
    }
    // LDS byte of the fragments 0, 4, .. (q = 0), .. of k-step ks of the stage at LDS byte `slot` (form N: of all
    // of them, q = 0); opaque, so that the fragments are reached by the reads' constant offsets from here
    __device__ __forceinline__ unsigned base(int q, int ks, unsigned slot) const
    {
        unsigned at = T ? rd[q % (T ? 4 : 2)] + slot : rd[ks] + slot;
        asm volatile("" : "+v"(at));
        return at;
    }
    // fragment i of the wave (16 rows x 32 k: lane l holds row l % 16, k = 8 (l / 16) .. + 7) of k-step ks; at:
    // base(i % 4 (form N: 0), ks, the stage's slot)
    __device__ __forceinline__ bf16x8 frag(int i, int ks, unsigned at) const
    {
        if constexpr (T) {
            typedef short short4v __attribute__((ext_vector_type(4)));
            typedef short short8v __attribute__((ext_vector_type(8)));
            typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
            at += PANEL * (unsigned)(i >> 2) + 4096u * (unsigned)ks;
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)at);
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(at + 512u));
            const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        } else {
            typedef __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
            return fpdt::as_bf16x8(*(lds_u32x4_ptr)(uintptr_t)(at + 2048u * (unsigned)i));
        }
    }
};

// A finished accumulator tile in ordinary registers.  The compiler does not know that the MFMAs are MFMAs, so it must
// not move an accumulator by itself (it would not wait for the result): behind the last MFMA they are read here and
// nowhere else, by statements that stay behind the wait.  (The last instruction: VALU results need two wait
// states before a lane exchange reads them, which the compiler does not see either.)
__device__ __forceinline__ floatx4 read_accumulator(const floatx4& acc)
{
    float x, y, z, w;
    asm volatile("v_accvgpr_read_b32 %0, %4\n\tv_accvgpr_read_b32 %1, %5\n\tv_accvgpr_read_b32 %2, %6\n\tv_accvgpr_read_b32 %3, %7\n\ts_nop 1"
                 : "=&v"(x), "=&v"(y), "=&v"(z), "=&v"(w)
                 : "a"(acc[0]), "a"(acc[1]), "a"(acc[2]), "a"(acc[3]));
    return floatx4{x, y, z, w};
}

// f(0), f(1), .. with the index as a constant of its type
template <int... I, typename F>
__device__ __forceinline__ void for_each_index(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

// C [M, N] row-major, leading dimension ldc elements.  A workgroup of four waves, one per SIMD, computes a
// (64 WMT) x (64 WNT) tile over the stages of its split; wave (w / 2, w % 2) owns 2 WMT x 2 WNT accumulator
// tiles of 16 x 16.
//
// What bounds it: the matrix cores are busy in 0.82, 0.79 and 0.73 of the cycles (8192^3, X W^T, dY W, dY^T X +=; nine tenths of
// the main loop's) at a clock that the power budget holds at 1.6-1.7 GHz, where the same loop without its copies runs at 1.9 and on registers alone at 2.0.
// The 128 x 128 elements of a wave at WMT = WNT = 4 need 16 KiB of fragments per 32 k (eight waves of 128 x 64: 24 KiB
// each pair).  The 256 accumulator registers leave room for one wave per SIMD, so nothing but this wave's own
// instruction order hides a latency.  A stage is two k-steps; the fragments of a k-step are read into a set of registers
// of their own under the MFMAs of the one before it.  The copies of stage s + 2 go out one at a time between the MFMAs
// of stage s: A's part, for which LDS has a third slot, in the first half, B's part in the second, into the slot that
// stage s has left.  One barrier per stage, between the halves: there stage s + 1 has landed and every wave has read all
// of stage s.
//
// Measured (8192^3 on cards where a library product takes 705-720 us; X W^T, dY W, dY^T X +=, us): stages of 32 k in
// four slots, whose copies read 64 bytes of a row of form N, 846, 857, 886; this 734, 712, 760: whole lines 765, 750,
// 808, the copies spread over the stage 751, 736, 765 (in half of its second half: 790, 775, 835), the bf16 epilogue
// straight from the accumulators (below) the rest.  16384 x 8192 x 8192: 1672, 1688, 1714 -> 1396, 1428, 1471.  Conflicts
// of form N's reads (half of their cycles with q ^ r % 8 ^ (r / 8) % 2 for a swizzle) cost nothing here.  With the
// 32 x 32 x 16 MFMA, which moves twice the accumulator registers per product, the loop took 6% more.  Operands packed
// into MFMA fragments first gave the loop 5-10% and cost 8-15% of an operation in packing.
//
// The MFMAs are issued through inline assembly so that the accumulators stay in accumulation registers
// for the whole loop (with the builtin the allocator moved tiles between the two register files).
// (B's fragment is the first operand: a lane then holds four consecutive columns of one row of C.)
#define TW_MFMA(d, x, y) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(y), "v"(x))
template <bool TA, bool TB, bool OUT_F32, bool ACCUM, int WMT, int WNT>
__global__ __launch_bounds__(NTHREAD, 1) void tw_gemm_kernel(Operand A, Operand B, int K, void* __restrict__ Cout, int64_t ldc,
                                                              int M, int N, Units u, float* __restrict__ part)
{
    // LDS: slots of a stage each, three of A and two of B.  64 x 256 tiles: two of each, so that two workgroups fit a
    // compute unit as with 128 x 128 (one runs its MFMAs under the other's first copies and its epilogue).
    constexpr bool SPREAD = WMT > 1;  // A's copies go out in the first half of a stage, into the third slot
    constexpr unsigned SLOT_A = WMT * PANEL, SLOT_B = WNT * PANEL, B0 = (SPREAD ? 3 : 2) * SLOT_A, LDS_BYTES = B0 + 2 * SLOT_B;
    constexpr int MI = 2 * WMT, NI = 2 * WNT;                   // accumulator tiles of a wave
    constexpr int NCA = 2 * WMT, NCB = 2 * WNT;                 // copies of a wave per stage
    static_assert(NWAVE == 4, "a wave copies a quarter of every panel");
    __shared__ __attribute__((aligned(256))) u32x4 ring[LDS_BYTES / 16];
    // Consecutive workgroup ids land on different XCDs (each with its own L2): give every XCD a
    // contiguous run of tiles, so that the tiles that share an operand row share an L2.  The units of the
    // divided tiles go half in front of the whole tiles and half behind them: the compute units that
    // start with one are out of step with the others from then on, and the epilogues of the ones run under
    // the MFMAs of the others.
    const unsigned xcd = blockIdx.x % 8, turn = blockIdx.x / 8;
    const unsigned divided = (unsigned)(u.tiles - u.whole), parts = divided * (unsigned)u.splits;
    const unsigned whole_run = ((unsigned)u.whole + 7) / 8, part_run = (parts + 7) / 8, lead = part_run / 2;
    const bool is_part = turn < lead || turn >= lead + whole_run;
    unsigned id = xcd * whole_run + turn - lead, split = 0;
    if (is_part) {
        const unsigned i = turn < lead ? turn : turn - whole_run, unit = xcd * part_run + i;
        if (i >= part_run || unit >= parts) return;  // whole workgroup, before any barrier
        id = (unsigned)u.whole + unit % divided;
        split = unit / divided;
    } else if (id >= (unsigned)u.whole) {
        return;
    }
    // Within a run the tiles go in groups of four tile rows, row index fastest: the 32 workgroups
    // that an XCD runs at a time then cover about 4 x 8 tiles and share 4 + 8 operand slices in its
    // L2 instead of 1 + 32.
    constexpr unsigned GROUP_M = 4;
    const unsigned tiles_n = (unsigned)u.tiles_n, tiles_m = (unsigned)u.tiles / tiles_n;
    const unsigned grp = id / (GROUP_M * tiles_n), in_grp = id % (GROUP_M * tiles_n);
    const unsigned rows_in_grp = tiles_m - grp * GROUP_M < GROUP_M ? tiles_m - grp * GROUP_M : GROUP_M;
    const int tile_m = (int)(grp * GROUP_M + in_grp % rows_in_grp), tile_n = (int)(in_grp / rows_in_grp);

    const int lane = threadIdx.x & 63;
    const int wu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wu >> 1, wn = wu & 1;
    const int stages = K / STAGE_K;  // whole ones
    const int unit_stages = is_part ? u.split_stages : stages, stage0 = (int)split * unit_stages;
    const int n_full = stages - stage0 < unit_stages ? stages - stage0 : unit_stages;
    const int k_left = stage0 + n_full == stages ? K % STAGE_K : 0;  // the last split's stage of less than STAGE_K
    const int total = n_full + (k_left > 0 ? 1 : 0);            // >= 1 (host)

    const unsigned ring0 = fpdt::lds_address(ring);
    Side<TA, WMT> a_side;
    Side<TB, WNT> b_side;
    a_side.init(A, tile_m * (64 * WMT), stage0, wu, wm * MI, lane, ring0);
    b_side.init(B, tile_n * (64 * WNT), stage0, wu, wn * NI, lane, ring0);
    const unsigned copy_lds = ring0 + 1024u * (unsigned)wu;
    // Copy j of a side's stage into the slot at LDS byte `slot_lds`: two scalar instructions besides the copy, the
    // second one for copy_address_rule (mfma_tiles.h) and as m0's wait state.
    auto copy = [](int j, unsigned off, uint64_t at, unsigned slot_lds) {
        uint64_t addr;
        asm volatile("s_add_u32 m0, %1, %2\n\ts_mov_b64 %0, %4\n\tglobal_load_lds_dwordx4 %3, %0"
                     : "=&s"(addr)
                     : "s"(slot_lds), "i"(PANEL * (j / 2) + 4096 * (j % 2)), "v"(off), "s"(at)
                     : "memory", "scc");
    };
    auto copy_a = [&](int j, unsigned slot_lds) { copy(j, a_side.off[j % 2][j / 2 % WMT], a_side.pos + (j % 2 ? a_side.half : 0), slot_lds); };
    auto copy_b = [&](int j, unsigned slot_lds) { copy(j, b_side.off[j % 2][j / 2 % WNT], b_side.pos + (j % 2 ? b_side.half : 0), slot_lds); };
    auto turn_to_tail = [&] {
        a_side.turn_to_tail(A, k_left, wu, lane);
        b_side.turn_to_tail(B, k_left, wu, lane);
    };
    auto clear_tail = [&](unsigned a_slot, unsigned b_slot) {  // (this wave's own copies have landed)
        a_side.clear_tail(k_left, wu, lane, copy_lds + a_slot);
        b_side.clear_tail(k_left, wu, lane, copy_lds + b_slot);
    };

    floatx4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+a"(acc[i][j]));
        }

    // the first two stages
    auto first_copies = [&](unsigned stage) {
#pragma unroll
        for (int j = 0; j < NCA; ++j) copy_a(j, copy_lds + stage * SLOT_A);
#pragma unroll
        for (int j = 0; j < NCB; ++j) copy_b(j, copy_lds + B0 + stage * SLOT_B);
    };
    if (n_full == 0) turn_to_tail();
    first_copies(0);
    if (total > 1) {
        a_side.pos += a_side.step;
        b_side.pos += b_side.step;
        if (n_full == 1) turn_to_tail();
        first_copies(1);
        fpdt::wait_vmem_at_most<NCA + NCB>();
    } else {
        fpdt::wait_vmem_at_most<0>();
        if (n_full == 0) clear_tail(0, B0);
    }
    fpdt::barrier_no_fence();

    bf16x8 a[2][MI], b[2][NI];  // by k-step
#pragma unroll
    for (int j = 0; j < NI; ++j) b[0][j] = b_side.frag(j, 0, b_side.base(TB ? j % 4 : 0, 0, B0));
#pragma unroll
    for (int i = 0; i < MI; ++i) a[0][i] = a_side.frag(i, 0, a_side.base(TA ? i % 4 : 0, 0, 0u));

    // Half of a stage: the MFMAs of k-step ks and, evenly between them, the fragments of the k-step behind it (of
    // the slots at LDS bytes a_slot and b_slot) and, with COPY, the copies of a stage: of A into the slot at `a_lds` in
    // the first half (SPREAD), of B into that at `b_lds` in the second.  (All of a stage's copies in its second half: 2%
    // slower; in half of that: 5%.)
    auto half_stage = [&](auto ks_tag, auto copy_tag, unsigned a_slot, unsigned b_slot, unsigned a_lds, unsigned b_lds) {
        constexpr int ks = decltype(ks_tag)::value, nx = 1 - ks;
        constexpr bool COPY = decltype(copy_tag)::value;
        constexpr int NM = MI * NI, NR = MI + NI;  // MFMAs, fragments
        constexpr int A_HERE = SPREAD == (ks == 0) ? NCA : 0, NC = A_HERE + (ks == 1 ? NCB : 0);  // copies
        constexpr int READ_SPAN = NM * 3 / 4;  // MFMAs over which the reads are spread: the last ones are not waited for
        unsigned a_at[4], b_at[4];
        for_each_index(std::make_integer_sequence<int, NM>{}, [&](auto m_tag) __attribute__((always_inline)) {
            constexpr int m = decltype(m_tag)::value;
            TW_MFMA(acc[m / NI][m % NI], a[ks][m / NI], b[ks][m % NI]);
            constexpr int r = (m * NR + READ_SPAN - 1) / READ_SPAN;
            if constexpr (m < READ_SPAN && r * READ_SPAN < (m + 1) * NR) {  // fragments in the order of their use
                if constexpr (r < NI) {
                    if (r < (TB ? 4 : 1)) b_at[r % 4] = b_side.base(r, nx, b_slot);
                    b[nx][r] = b_side.frag(r, nx, b_at[TB ? r % 4 : 0]);
                } else {
                    if (r - NI < (TA ? 4 : 1)) a_at[(r - NI) % 4] = a_side.base(r - NI, nx, a_slot);
                    a[nx][r - NI] = a_side.frag(r - NI, nx, a_at[TA ? (r - NI) % 4 : 0]);
                }
            }
            constexpr int c = (m * NC + NM - 1) / NM;
            if constexpr (COPY && c * NM < (m + 1) * NC) {
                if constexpr (c < A_HERE) copy_a(c, a_lds);
                else copy_b(c - A_HERE, b_lds);
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        static_assert(NR <= READ_SPAN && NC <= NM, "at most one of each behind an MFMA");
    };
    typedef std::integral_constant<int, 0> Ks0;
    typedef std::integral_constant<int, 1> Ks1;
    // slots (LDS bytes) of the current stage s, of stage s + 1, and of A's part of stage s + 2 (its part of B takes the
    // slot of stage s)
    unsigned cur_a = 0, cur_b = B0, nxt_a = SLOT_A, nxt_b = B0 + SLOT_B, free_a = SPREAD ? 2 * SLOT_A : 0;
    auto next_stage = [&] {
        const unsigned was_a = cur_a, was_b = cur_b;
        cur_a = nxt_a;
        cur_b = nxt_b;
        nxt_a = free_a;
        nxt_b = was_b;
        free_a = SPREAD ? was_a : cur_a;
    };
    // the stages behind the first two: the whole ones, then the last one of less than STAGE_K
    int copied = n_full > 2 ? n_full - 2 : 0;
#pragma unroll 1
    for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
        for (; copied > 0; --copied) {
            a_side.pos += a_side.step;
            b_side.pos += b_side.step;
            half_stage(Ks0{}, std::true_type{}, cur_a, cur_b, copy_lds + free_a, 0u);
            fpdt::wait_vmem_at_most<SPREAD ? NCA : 0>();  // the next stage: all but the copies just issued
            fpdt::barrier_no_fence();  // everyone's part of it; everyone has read all of this one
            __builtin_amdgcn_sched_barrier(0);
            half_stage(Ks1{}, std::true_type{}, nxt_a, nxt_b, copy_lds + free_a, copy_lds + cur_b);
            next_stage();
        }
        if (pass == 0 && k_left > 0 && n_full >= 2) {
            a_side.pos += a_side.step;
            b_side.pos += b_side.step;
            turn_to_tail();
            copied = 1;
        }
    }
    // the last two
    int left = total < 2 ? total : 2;
    do {
        half_stage(Ks0{}, std::false_type{}, cur_a, cur_b, 0u, 0u);
        fpdt::wait_vmem_at_most<0>();
        if (left == 2 && k_left > 0) clear_tail(nxt_a, nxt_b);
        fpdt::barrier_no_fence();
        __builtin_amdgcn_sched_barrier(0);
        half_stage(Ks1{}, std::false_type{}, nxt_a, nxt_b, 0u, 0u);  // (behind the last stage: fragments of idle slots, not used)
        next_stage();
    } while (--left > 0);
    fpdt::barrier_no_fence();  // nobody reads the ring any more

    // the accumulators are read by ordinary instructions from here on
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    // accumulator tile (i, j): lane l holds row l % 16, columns 4 (l / 16) .. + 3
    const int mw = wm * (32 * WMT), nw = wn * (32 * WNT);  // the wave's first row and column within the tile
    // `m_left`, `n_left` below: rows and columns of C from `out` on; where they end within the tile, they end with
    // 16 bytes (WHOLE: they do not, and no access is conditional: conditional loads of old values wait for each
    // other, 8192^3, dY^T X, 800 -> 890 us).  With ACC the old values of sixteen rows are all requested, and those of the next sixteen in front of
    // their stores: one load at a time, each waited for behind the store before it, left the read-modify-write of a
    // weight gradient at a sixth of the memory rate.
    //
    // fp32: sixteen rows at a time pass through LDS (each wave its own part of the idle ring), so that an access
    // covers 128 WNT bytes of a row.  This is bound by the memory: 14 us per tile of 256 x 256 added to, of all
    // compute units.  (Straight from the accumulators, 64 bytes of sixteen rows or 128 of eight per access: 8192^3,
    // dY^T X, 779 -> 830 and 860 us.)
    auto store_f32 = [&](float* out, int64_t pitch, int m_left, int n_left, auto acc_tag, auto whole_tag) {
        constexpr bool ACC = decltype(acc_tag)::value, WHOLE = decltype(whole_tag)::value;
        constexpr int LPR = 8 * WNT, RPI = 64 / LPR, PITCH = 32 * WNT + 4;  // lanes per row, rows per access, floats (4 apart: no bank conflicts)
        static_assert(4 * 16 * PITCH * 4 <= (int)LDS_BYTES, "the ring holds sixteen rows of every wave");
        float* rows = reinterpret_cast<float*>(ring) + wu * (16 * PITCH);
        float* put = rows + (lane & 15) * PITCH + 4 * (lane >> 4);
        const float* get = rows + (lane / LPR) * PITCH + 4 * (lane % LPR);
        const int row = mw + lane / LPR, col = nw + 4 * (lane % LPR);
        float* c0 = out + (int64_t)row * pitch + col;
        auto in = [&](int i, int k) { return WHOLE || (row + 16 * i + RPI * k < m_left && col < n_left); };
        floatx4 old[2][NI];
        auto request = [&](int i) {
#pragma unroll
            for (int k = 0; k < NI; ++k)
                if (in(i, k)) old[i & 1][k] = *reinterpret_cast<const floatx4*>(c0 + (int64_t)(16 * i + RPI * k) * pitch);
        };
        if (ACC) request(0);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (ACC && i + 1 < MI) request(i + 1);
            __builtin_amdgcn_sched_barrier(0);  // no further ahead: the registers are spoken for
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                *reinterpret_cast<floatx4*>(put + 16 * j) = read_accumulator(acc[i][j]);
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                floatx4 v = *reinterpret_cast<const floatx4*>(get + RPI * k * PITCH);
                if (ACC) v = old[i & 1][k] + v;
                if (in(i, k)) *reinterpret_cast<floatx4*>(c0 + (int64_t)(16 * i + RPI * k) * pitch) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
    // bf16: straight from the accumulators, 16 bytes per lane and access.  Two neighbouring tiles exchange lane groups,
    // so that group g holds columns 8 (g / 2) .. + 7 of tile j + g % 2: an access covers 64 bytes of sixteen rows.
    // (Through LDS, and rounded in integer arithmetic, a tile of 256 x 256 took 17 us, during which the matrix
    // cores idle: 8192^3, X W^T, 755 -> 738 us.  128 bytes of eight rows per access: the same.)
    auto store_bf16 = [&](uint16_t* out, int64_t pitch, int m_left, int n_left, auto acc_tag, auto whole_tag) {
        constexpr bool ACC = decltype(acc_tag)::value, WHOLE = decltype(whole_tag)::value;
        constexpr int NA = NI / 2;
        const int g = lane >> 4, row = mw + (lane & 15), col = nw + 16 * (g & 1) + 8 * (g >> 1);
        uint16_t* c0 = out + (int64_t)row * pitch + col;
        auto in = [&](int i, int k) { return WHOLE || (row + 16 * i < m_left && col + 32 * k < n_left); };
        u32x4 old[2][NA];
        auto request = [&](int i) {
#pragma unroll
            for (int k = 0; k < NA; ++k)
                if (in(i, k)) old[i & 1][k] = *reinterpret_cast<const u32x4*>(c0 + (int64_t)(16 * i) * pitch + 32 * k);
        };
        if (ACC) request(0);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (ACC && i + 1 < MI) request(i + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < NA; ++k) {
                const floatx4 a0 = read_accumulator(acc[i][2 * k]), a1 = read_accumulator(acc[i][2 * k + 1]);
                u32x4 v;
                if constexpr (!ACC) {
                    const u32x4 x = pack_bf16(a0, a1);
                    const auto lo = __builtin_amdgcn_permlane16_swap(x[0], x[2], false, false);
                    const auto hi = __builtin_amdgcn_permlane16_swap(x[1], x[3], false, false);
                    v = u32x4{lo[0], hi[0], lo[1], hi[1]};
                } else {  // exchanged in fp32, as they are added to before they are rounded
                    const u32x4 o = old[i & 1][k];
                    floatx4 x, y;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const auto xy = __builtin_amdgcn_permlane16_swap(__float_as_uint(a0[r]), __float_as_uint(a1[r]), false, false);
                        x[r] = __uint_as_float((o[r / 2] << (r % 2 ? 0 : 16)) & 0xffff0000u) + __uint_as_float(xy[0]);
                        y[r] = __uint_as_float((o[2 + r / 2] << (r % 2 ? 0 : 16)) & 0xffff0000u) + __uint_as_float(xy[1]);
                    }
                    v = pack_bf16(x, y);
                }
                if (in(i, k)) *reinterpret_cast<u32x4*>(c0 + (int64_t)(16 * i) * pitch + 32 * k) = v;
            }
        }
    };
    if (is_part) {  // this split's sums of the whole tile; tw_split_sum_kernel adds them
        constexpr size_t TILE_ELEMS = (size_t)(64 * WMT) * (64 * WNT);
        store_f32(part + ((size_t)split * divided + (id - (unsigned)u.whole)) * TILE_ELEMS, 64 * WNT, 64 * WMT, 64 * WNT, std::false_type{}, std::true_type{});
        return;
    }
    typedef typename std::conditional<OUT_F32, float, uint16_t>::type out_t;
    const int mt = tile_m * (64 * WMT), nt = tile_n * (64 * WNT);
    out_t* tile = static_cast<out_t*>(Cout) + (size_t)mt * ldc + nt;
    constexpr int PER16 = 16 / sizeof(out_t);
    // (fp32, not added to: rows that are not a multiple of four long but that far apart end with room for one, tw_gemm.h)
    if ((N % PER16 == 0 || (OUT_F32 && !ACCUM)) && ldc % PER16 == 0 && reinterpret_cast<uintptr_t>(Cout) % 16 == 0) {
        auto store = [&](auto whole_tag) {
            if constexpr (OUT_F32) store_f32(tile, ldc, M - mt, N - nt, std::integral_constant<bool, ACCUM>{}, whole_tag);
            else store_bf16(tile, ldc, M - mt, N - nt, std::integral_constant<bool, ACCUM>{}, whole_tag);
        };
        if (mt + 64 * WMT <= M && nt + 64 * WNT <= N) store(std::true_type{});
        else store(std::false_type{});
        return;
    }
    // Rows of C that do not come in pieces of 16 bytes: sixteen rows at a time through LDS (each wave its own part
    // of the idle ring), one element per lane and access, consecutive lanes on consecutive columns.  (Straight
    // from the accumulators an access touched 16 rows at 16 bytes each: odd widths then took up to twice the
    // time of the tiles' MFMAs.)  The old values of the sixteen rows are requested together.
    constexpr int PITCH = 32 * WNT + 4, CPR = 32 * WNT / 64;  // floats between rows (4 apart: no bank conflicts), accesses per row
    static_assert(4 * 16 * PITCH * 4 <= (int)LDS_BYTES, "the ring holds sixteen rows of every wave");
    float* rows = reinterpret_cast<float*>(ring) + wu * (16 * PITCH);
    float* put = rows + (lane & 15) * PITCH + 4 * (lane >> 4);
    bool in[CPR];
#pragma unroll
    for (int p = 0; p < CPR; ++p) in[p] = nt + nw + 64 * p + lane < N;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int left = M - (mt + mw + 16 * i);  // rows of C from here on
        if (left <= 0) break;
        out_t* c = tile + (size_t)(mw + 16 * i) * ldc + nw + lane;
        out_t old[16][CPR];
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int p = 0; p < CPR; ++p) old[r][p] = ACCUM && r < left && in[p] ? c[(size_t)r * ldc + 64 * p] : out_t(0);
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            *reinterpret_cast<floatx4*>(put + 16 * j) = read_accumulator(acc[i][j]);
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int p = 0; p < CPR; ++p)
                if (r < left && in[p]) c[(size_t)r * ldc + 64 * p] = combine<ACCUM>(rows[r * PITCH + 64 * p + lane], old[r][p]);
        __builtin_amdgcn_wave_barrier();
    }
}

// The divided tiles of a product: C (+)= the sums of their splits, part [split][tile][TM x TN] fp32.
// Memory-bound: (splits + 1) passes over those tiles.
template <bool OUT_F32, bool ACCUM>
__global__ __launch_bounds__(256) void tw_split_sum_kernel(const float* __restrict__ part, Units u, int first, int tm, int tn, void* __restrict__ Cout,
                                                            int64_t ldc, int M, int N)
{
    typedef typename std::conditional<OUT_F32, float, uint16_t>::type out_t;
    typedef out_t out4 __attribute__((ext_vector_type(4)));
    constexpr unsigned GROUP_M = 4;  // the order of the tiles, as in the product
    const unsigned i = (unsigned)first + blockIdx.y, id = (unsigned)u.whole + i, tiles_n = (unsigned)u.tiles_n, tiles_m = (unsigned)u.tiles / tiles_n;
    const unsigned grp = id / (GROUP_M * tiles_n), in_grp = id % (GROUP_M * tiles_n);
    const unsigned rows_in_grp = tiles_m - grp * GROUP_M < GROUP_M ? tiles_m - grp * GROUP_M : GROUP_M;
    const int tile_m = (int)(grp * GROUP_M + in_grp % rows_in_grp), tile_n = (int)(in_grp / rows_in_grp);
    const int at = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4;  // within the tile: tm * tn is a multiple of 1024
    const int m = tile_m * tm + at / tn, n = tile_n * tn + at % tn;
    if (m >= M || n >= N) return;
    const size_t stride = (size_t)(u.tiles - u.whole) * tm * tn;
    const float* p = part + (size_t)i * tm * tn + at;
    floatx4 v = *reinterpret_cast<const floatx4*>(p);
    for (int s = 1; s < u.splits; ++s) v += *reinterpret_cast<const floatx4*>(p + s * stride);
    out_t* c = static_cast<out_t*>(Cout) + (size_t)m * ldc + n;
    if (n + 4 <= N && ldc % 4 == 0 && reinterpret_cast<uintptr_t>(Cout) % (4 * sizeof(out_t)) == 0) {
        out4 o = {};
        if (ACCUM) o = *reinterpret_cast<const out4*>(c);
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = combine<ACCUM>(v[r], o[r]);
        *reinterpret_cast<out4*>(c) = o;
    } else {
        for (int r = 0; r < 4 && n + r < N; ++r) c[r] = combine<ACCUM>(v[r], ACCUM ? c[r] : out_t(0));
    }
}

// ---- host side: scratch and the per-call cache of realigned weights --------------
struct Pool {
    char* base = nullptr;
    size_t cap = 0, off = 0;
    std::vector<void*> retired;  // outgrown buffers: work already enqueued may still read them
};
struct Realigned {
    const void* src;
    int64_t R, C, ld;
    const uint16_t* copy;
};
Pool g_pool[64];
std::vector<Realigned> g_cache;  // weights realigned during the current library call
std::mutex g_mu;

int pool_take(Pool& p, size_t bytes, char** out)
{
    bytes = (bytes + 255) & ~(size_t)255;
    if (p.off + bytes > p.cap) {
        // Grow: a new buffer; the old one stays alive (kernels in flight, and the rest of this call, read
        // it) until exit.  The call's offsets go on as if all of it were in the new buffer, so that it
        // holds all of the next call of these sizes, which may be captured.
        size_t want = p.cap ? p.cap * 2 : (size_t)256 << 20;
        while (want < p.off + bytes) want *= 2;
        void* nb = nullptr;
        if (hipMalloc(&nb, want) != hipSuccess) {
            (void)hipGetLastError();
            return 1;
        }
        if (p.base) p.retired.push_back(p.base);
        p.base = static_cast<char*>(nb);
        p.cap = want;
    }
    *out = p.base + p.off;
    p.off += bytes;
    return 0;
}

// A lane's offset within its tile (255 rows of form N, 7 of form T) is kept in 32 bits
constexpr int64_t MAX_PITCH = (int64_t)1 << 23;    // elements between rows along k
constexpr int64_t MAX_PITCH_T = (int64_t)1 << 28;  // and between the rows of k, form T
constexpr int64_t COPY_PAD = 64;                   // a copy's rows are this many elements further apart at most

// The bytes that a product writes
struct Written {
    const void* C;
    int64_t rows, cols, ld;
    int size;
    bool overlaps(const void* X, int64_t R, int64_t cols_x, int64_t ld_x) const
    {
        const uintptr_t c = reinterpret_cast<uintptr_t>(C), x = reinterpret_cast<uintptr_t>(X);
        return x < c + (uintptr_t)((rows - 1) * ld + cols) * size && c < x + (uintptr_t)((R - 1) * ld_x + cols_x) * 2;
    }
};

// Can the product kernel read X [R, C] where it is?
bool readable(const void* X, int64_t R, int64_t C, int64_t ld, bool k_rows, bool padded, const Written& out)
{
    return (C % 8 == 0 || padded) && ld % 8 == 0 && ld < (k_rows ? MAX_PITCH_T : MAX_PITCH) &&
           reinterpret_cast<uintptr_t>(X) % 16 == 0 && !out.overlaps(X, R, C, ld);
}

// X [R, C], leading dimension ld, as the product kernel can read it: in place, or copied.  `k_rows`: the
// contraction runs over the rows of X.  `padded`: rows are followed by zeros up to a multiple of 8.
// An operand that the product itself overwrites (Y in the place of X) is copied: tiles are stored while
// others still read their rows.
int take_operand(Pool& pool, const void* X, int64_t R, int64_t C, int64_t ld, bool k_rows, bool padded, bool cache, const Written& out,
                 hipStream_t st, Operand* res)
{
    res->rows = (int)(k_rows ? (C + 7) / 8 * 8 : R);
    if (readable(X, R, C, ld, k_rows, padded, out)) {
        res->p = static_cast<const uint16_t*>(X);
        res->ld = ld;
    } else {
        const int64_t C2 = (C + 7) / 8 * 8;
        // whole cache lines from row to row: a stage's part of a row is a line (form N: 64 k, form T: 64 columns), and with
        // 8208 bytes from row to row in place of 8320 it lay in two (Y of 16384 x 4097 x 4096: 493 -> 451 us, in 8 chunks
        // 626 -> 542)
        res->ld = C2 <= 64 ? C2 : (C2 + 63) / 64 * 64;
        res->p = nullptr;
        if (cache)
            for (const Realigned& c : g_cache)
                if (c.src == X && c.R == R && c.C == C && c.ld == ld) res->p = c.copy;
        if (!res->p) {
            char* mem = nullptr;
            if (pool_take(pool, (size_t)R * res->ld * 2, &mem)) return 1;
            const int64_t blocks = (R * (C2 / 8) + 255) / 256;
            tw_realign_kernel<<<dim3((unsigned)(blocks < 65536 ? blocks : 65536)), 256, 0, st>>>(
                static_cast<const uint16_t*>(X), R, C, ld, reinterpret_cast<u32x4*>(mem), res->ld);
            res->p = reinterpret_cast<const uint16_t*>(mem);
            if (cache) g_cache.push_back({X, R, C, ld, res->p});
        }
    }
    return res->ld >= (k_rows ? MAX_PITCH_T : MAX_PITCH) ? 2 : 0;
}

}  // namespace

void begin_call()
{
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
    g_cache.clear();
    g_pool[dev].off = 0;  // everything enqueued earlier on the stream is ordered before what follows
}

bool reads_in_place(const void* A, int64_t rows, int64_t k, const void* C, int64_t cols)
{
    return readable(A, rows, k, k, false, false, Written{C, rows, cols, cols, 2});
}

void* scratch(size_t bytes)
{
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    char* mem = nullptr;
    return pool_take(g_pool[dev], bytes, &mem) ? nullptr : mem;
}

// The launch of a product (or, with u.whole = 0 and one split at a time, of one k segment of it)
static int launch_product(const Plan& plan, int a_transposed, int b_transposed, const Operand& a, const Operand& b, int M, int N, int K,
                          void* C, int64_t ldc, bool c_f32, bool accumulate, float* part, hipStream_t st)
{
    const Units& u = plan.u;
    const int64_t parts = (int64_t)(u.tiles - u.whole) * u.splits;
    const unsigned grid = 8 * ((unsigned)((u.whole + 7) / 8) + (unsigned)((parts + 7) / 8));
#define TW_LAUNCH_TILE(TA, TB, F32, ACC, WM, WN) tw_gemm_kernel<TA, TB, F32, ACC, WM, WN><<<grid, NTHREAD, 0, st>>>(a, b, K, C, ldc, M, N, u, part)
#define TW_LAUNCH(TA, TB, F32, ACC)                                             \
    do {                                                                        \
        if (plan.wnt == 2) TW_LAUNCH_TILE(TA, TB, F32, ACC, 2, 2);              \
        else if (plan.wmt == 4) TW_LAUNCH_TILE(TA, TB, F32, ACC, 4, 4);         \
        else if (plan.wmt == 3) TW_LAUNCH_TILE(TA, TB, F32, ACC, 3, 4);         \
        else if (plan.wmt == 2) TW_LAUNCH_TILE(TA, TB, F32, ACC, 2, 4);         \
        else TW_LAUNCH_TILE(TA, TB, F32, ACC, 1, 4);                            \
    } while (0)
    // the forms and outputs that the library's operations use
    if (!a_transposed && !b_transposed && !accumulate) {
        if (c_f32) TW_LAUNCH(false, false, true, false);
        else TW_LAUNCH(false, false, false, false);
    } else if (!a_transposed && b_transposed && !c_f32) {
        if (accumulate) TW_LAUNCH(false, true, false, true);
        else TW_LAUNCH(false, true, false, false);
    } else if (a_transposed && b_transposed && c_f32 && accumulate) {
        TW_LAUNCH(true, true, true, true);
    } else {
        return 2;
    }
#undef TW_LAUNCH
#undef TW_LAUNCH_TILE
    return 0;
}

static size_t part_bytes(const Plan& plan) { return (size_t)plan.u.splits * (plan.u.tiles - plan.u.whole) * (64 * plan.wmt) * (64 * plan.wnt) * 4; }

static void launch_split_sum(const Plan& plan, const float* part, int M, int N, void* C, int64_t ldc, bool c_f32, bool accumulate, hipStream_t st)
{
    const int tm = 64 * plan.wmt, tn = 64 * plan.wnt, divided = plan.u.tiles - plan.u.whole;
    for (int t0 = 0; t0 < divided; t0 += 65535) {  // the grid's second dimension
        const Units& u = plan.u;
        const dim3 grid((unsigned)(tm * tn / 1024), (unsigned)(divided - t0 < 65535 ? divided - t0 : 65535));
        if (c_f32 && accumulate) tw_split_sum_kernel<true, true><<<grid, 256, 0, st>>>(part, u, t0, tm, tn, C, ldc, M, N);
        else if (c_f32) tw_split_sum_kernel<true, false><<<grid, 256, 0, st>>>(part, u, t0, tm, tn, C, ldc, M, N);
        else if (accumulate) tw_split_sum_kernel<false, true><<<grid, 256, 0, st>>>(part, u, t0, tm, tn, C, ldc, M, N);
        else tw_split_sum_kernel<false, false><<<grid, 256, 0, st>>>(part, u, t0, tm, tn, C, ldc, M, N);
    }
}

static int product(Pool& pool, int a_transposed, int b_transposed, int M, int N, int K, const void* A, int64_t lda, const void* B,
                   int64_t ldb, void* C, int64_t ldc, bool c_f32, bool accumulate, bool cache_b, hipStream_t st)
{
    const size_t off0 = pool.off;
    const Plan plan = plan_launch(M, N, (K < SK ? SK : K) / SK);
    if (plan.u.tiles == 0) return 2;
    // Aop[m,k]: A stored [M,K] (as is) or [K,M] (transposed); Bop[n,k]: B stored [N,K] or [K,N]
    const Written out = {C, M, N, ldc, c_f32 ? 4 : 2};
    Operand pa, pb;
    int rc = take_operand(pool, B, b_transposed ? K : N, b_transposed ? N : K, ldb, b_transposed, false, cache_b, out, st, &pb);
    if (rc) return rc;
    const size_t mark = pool.off;  // what follows is scratch of this product only
    rc = take_operand(pool, A, a_transposed ? K : M, a_transposed ? M : K, lda, a_transposed, lda > (a_transposed ? M : K), false, out, st, &pa);
    if (rc) return rc;
    float* part = nullptr;
    if (plan.u.splits > 1) {
        char* mem = nullptr;
        if (pool_take(pool, part_bytes(plan), &mem)) return 1;
        part = reinterpret_cast<float*>(mem);
    }
    rc = launch_product(plan, a_transposed, b_transposed, pa, pb, M, N, K, C, ldc, c_f32, accumulate, part, st);
    if (rc) return rc;
    if (plan.u.splits > 1) launch_split_sum(plan, part, M, N, C, ldc, c_f32, accumulate, st);
    // The next product's copies run after this launch on the same stream, so this product's scratch
    // is free again: everything it took, or everything behind a weight that stays cached.
    pool.off = cache_b ? mark : off0;
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

static int any_product(Pool& pool, int a_transposed, int b_transposed, int M, int N, int K, const void* A, int64_t lda, const void* B,
                       int64_t ldb, void* C, int64_t ldc, bool c_f32, bool accumulate, bool cache_b, hipStream_t st)
{
    // Rows of k too far apart (form T, an operand of more than 2^28 columns): the columns, which are rows or
    // columns of C, in segments, whose copies have a shorter pitch.  More than 2^30 columns of C in segments
    // too: the last tile would reach behind 2^31.
    constexpr int SEG_T = 1 << 24, SEG_N = 1 << 30;
    const int seg_n = b_transposed && ldb > MAX_PITCH_T - COPY_PAD ? SEG_T : SEG_N;
    if (N > seg_n) {
        for (int64_t n0 = 0; n0 < N; n0 += seg_n) {
            const int rc = any_product(pool, a_transposed, b_transposed, M, (int)(N - n0 < seg_n ? N - n0 : seg_n), K, A, lda,
                                       static_cast<const uint16_t*>(B) + (b_transposed ? n0 : n0 * ldb), ldb,
                                       static_cast<char*>(C) + n0 * (c_f32 ? 4 : 2), ldc, c_f32, accumulate, false, st);
            if (rc) return rc;
        }
        return 0;
    }
    if (a_transposed && lda > MAX_PITCH_T - COPY_PAD && M > SEG_T) {
        for (int64_t m0 = 0; m0 < M; m0 += SEG_T) {
            const int rc = any_product(pool, a_transposed, b_transposed, (int)(M - m0 < SEG_T ? M - m0 : SEG_T), N, K, static_cast<const uint16_t*>(A) + m0, lda, B, ldb,
                                       static_cast<char*>(C) + (size_t)m0 * ldc * (c_f32 ? 4 : 2), ldc, c_f32, accumulate, cache_b, st);
            if (rc) return rc;
        }
        return 0;
    }
    const bool long_a = !a_transposed && lda > MAX_PITCH - COPY_PAD, long_b = !b_transposed && ldb > MAX_PITCH - COPY_PAD;
    if (!long_a && !long_b)
        return product(pool, a_transposed, b_transposed, M, N, K, A, lda, B, ldb, C, ldc, c_f32, accumulate, cache_b, st);
    // Rows too long for the kernel's offsets: k in segments, which are the splits of every tile, one launch
    // each; the long operand's segment is copied out in front of it.
    constexpr int64_t SEG = (int64_t)1 << 22;
    Plan plan = {4, 4, {}};
    const int64_t tiles_n = ((int64_t)N + 255) / 256, tiles = ((int64_t)M + 255) / 256 * tiles_n;
    if (tiles > (int64_t)1 << 30) return 2;
    plan.u = {(int)tiles, (int)tiles_n, 0, (int)((K + SEG - 1) / SEG), 0};
    const size_t off0 = pool.off;
    char* mem = nullptr;
    if (pool_take(pool, part_bytes(plan), &mem)) return 1;
    float* part = reinterpret_cast<float*>(mem);
    for (int i = 0; i < plan.u.splits; ++i) {
        const int64_t k0 = i * SEG, k = K - k0 < SEG ? K - k0 : SEG;
        const size_t off1 = pool.off;
        Operand a, b;
        // (a segment of a long row is never read in place: its pitch is the row's; C is written behind all of them)
        const Written out = {part, 1, 1, 1, 4};
        int rc = take_operand(pool, static_cast<const uint16_t*>(B) + (b_transposed ? k0 * ldb : k0), b_transposed ? k : N, b_transposed ? N : k, ldb, b_transposed, false, false, out, st, &b);
        if (!rc) rc = take_operand(pool, static_cast<const uint16_t*>(A) + (a_transposed ? k0 * lda : k0), a_transposed ? k : M, a_transposed ? M : k, lda, a_transposed, false, false, out, st, &a);
        if (rc) return rc;
        Plan one = plan;
        one.u.splits = 1;
        one.u.split_stages = (int)(k / STAGE_K);
        rc = launch_product(one, a_transposed, b_transposed, a, b, M, N, (int)k, C, ldc, c_f32, accumulate, part + (size_t)i * (part_bytes(one) / 4), st);
        if (rc) return rc;
        pool.off = off1;
    }
    launch_split_sum(plan, part, M, N, C, ldc, c_f32, accumulate, st);
    pool.off = off0;
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

int gemm(int a_transposed, int b_transposed, int M, int N, int K, const void* A, int64_t lda, const void* B,
         int64_t ldb, void* C, int64_t ldc, bool c_f32, bool accumulate, bool cache_b, hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1;
    if (M <= 0 || N <= 0 || K <= 0) return 2;
    return any_product(g_pool[dev], a_transposed, b_transposed, M, N, K, A, lda, B, ldb, C, ldc, c_f32, accumulate, cache_b, st);
}

}  // namespace fpdt_tw
