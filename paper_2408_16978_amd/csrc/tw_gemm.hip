// Dense bf16 products of the token-wise chunked operations (Sec. 4.1, 5.4: the per-chunk QKV
// projection, the feed-forward block and the output projection of the loss are plain GEMMs over
// one chunk of tokens at a time) on v_mfma_f32_16x16x32_bf16: a four-slot LDS ring filled by direct
// global -> LDS copies three stages ahead, four waves (one per SIMD) per output tile of up to
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
// The product kernel copies 16-byte pieces of its operands' rows and needs at least one whole stage of
// k.  An operand that does not offer that (a width that is not a multiple of 8, a base that is not
// 16-byte aligned, k < 32), or that the product overwrites, is copied once into out [R2, C2], zero behind
// X [R, C], rows `pitch` elements apart.
__global__ __launch_bounds__(256) void tw_realign_kernel(const uint16_t* __restrict__ X, int64_t R, int64_t C, int64_t ld,
                                                         u32x4* __restrict__ out, int64_t R2, int64_t C2, int64_t pitch)
{
    const int64_t pieces = C2 / 8, n = R2 * pieces;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t r = n >> 32 ? i / pieces : (unsigned)i / (unsigned)pieces, c = (i - r * pieces) * 8;
        u32x4 v;
        if (r < R && c + 8 <= C) {  // (16 bytes at any even address in one access)
            __builtin_memcpy(&v, X + r * ld + c, 16);
        } else {
            unsigned e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = r < R && c + j < C ? X[r * ld + c + j] : 0u;
            v = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        }
        out[r * (pitch / 8) + c / 8] = v;
    }
}

// ---- product ----------------------------------------------------------------------------
constexpr int NWAVE = 4, NTHREAD = NWAVE * 64;
constexpr int RING = 4;       // LDS slots of one stage each; one more holds a last stage of less than SK
constexpr unsigned PANEL = 4096;  // bytes of a panel: 64 rows of one operand x SK

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
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
// rows; wave w copies quarter w of every panel.
//   Form N: panel row r (64 bytes) holds its four 16-byte pieces q at position q ^ f(r),
//           f(r) = (r / 2) % 4 ^ (r / 8) % 2: any 8 rows aligned to 8, read at one piece, lie in different
//           16-byte columns of 128 bytes, and any 16 rows in different columns of 256 bytes.
//   Form T: panel row k (128 bytes, 64 columns) holds its 32-byte quarter u at u ^ (2 ((k / 2) % 2) + (k / 8) % 2):
//           the eight k x 16 columns that half a wave's transposing read covers lie in different 32-byte
//           columns of 256 bytes.
template <bool T, int NP>
struct Side {
    uint64_t pos;        // scalar: the current stage
    uint64_t step;       // bytes from a stage to the next
    unsigned off[NP];    // this lane's piece of panel j
    unsigned rd[4];      // LDS bytes within a stage: of fragments 0, 4, .., of 1, 5, .., (form N: rd[0] only)

    __device__ __forceinline__ void init(const Operand& x, int row0, int stage0, int w, int wave_frag0, int lane, unsigned lds0)
    {
        const uint64_t pitch = (uint64_t)x.ld * 2;
        const int limit = x.rows - row0;  // >= 1
        if (T) {
            step = SK * pitch;
            pos = (uint64_t)(uintptr_t)(x.p + row0) + (uint64_t)stage0 * step + (uint64_t)(8 * w) * pitch;
            const int k = lane >> 3, u = ((lane >> 1) & 3) ^ (2 * ((k >> 1) & 1) + (w & 1));
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int c = 64 * j + 16 * u + 8 * (lane & 1);
                off[j] = (unsigned)k * (unsigned)pitch + 2u * (unsigned)(c < limit - 8 ? c : limit - 8);
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
            step = SK * 2;
            pos = (uint64_t)(uintptr_t)x.p + (uint64_t)row0 * pitch + (uint64_t)stage0 * step;
            const int r = lane >> 2, q = (lane & 3) ^ ((r >> 1) & 3) ^ ((r >> 3) & 1);
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                // rows behind the operand are read as its last row: their products are not stored
                const int mine = 64 * j + 16 * w + r < limit ? 64 * j + 16 * w + r : limit - 1;
                off[j] = (unsigned)mine * (unsigned)pitch + 16u * (unsigned)q;
            }
            const int fr = lane & 15, swz = ((fr >> 1) & 3) ^ ((fr >> 3) & 1);
            rd[0] = lds0 + 64u * (unsigned)(16 * wave_frag0 + fr) + 16u * (unsigned)((lane >> 4) ^ swz);
        }
        pos = fpdt::uniform(pos);
    }
    // does this lane's piece of stage `s` hold k < K (form N: K rounded up to 8)?
    __device__ __forceinline__ bool has(int s, int K, int w, int lane) const
    {
        if (T) return s * SK + 8 * w + (lane >> 3) < K;
        const int r = lane >> 2, q = (lane & 3) ^ ((r >> 1) & 3) ^ ((r >> 3) & 1);
        return s * SK + 8 * q < K;
    }
    // fragment i of the wave (16 rows x 32 k: lane l holds row l % 16, k = 8 (l / 16) .. + 7) of the stage at
    // LDS byte `slot`
    __device__ __forceinline__ bf16x8 frag(int i, unsigned slot) const
    {
        if (T) {
            typedef short short4v __attribute__((ext_vector_type(4)));
            typedef short short8v __attribute__((ext_vector_type(8)));
            typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
            const unsigned at = rd[i & 3] + slot + PANEL * (unsigned)(i >> 2);
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)at);
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(at + 512u));
            const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        }
        typedef __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
        return fpdt::as_bf16x8(*(lds_u32x4_ptr)(uintptr_t)(rd[0] + slot + 1024u * (unsigned)i));
    }
};

// C [M, N] row-major, leading dimension ldc elements.  A workgroup of four waves, one per SIMD, computes a
// (64 WMT) x (64 WNT) tile over the stages of its split; wave (w / 2, w % 2) owns 2 WMT x 2 WNT accumulator
// tiles of 16 x 16.
//
// What bounds it: LDS traffic next to the MFMAs.  The 128 x 128 elements of a wave at WMT = WNT = 4 need
// 16 KiB of fragments per 32 k; eight waves of 128 x 64 need 24 KiB each pair, and with the copies' writes
// LDS was then as busy as the MFMA pipes.  The 256 accumulator registers leave room for one wave per SIMD,
// so nothing but this wave's own instruction order hides a latency.  A stage runs in two phases, the left
// and the right half of the wave's columns.  Each fragment register is read again as soon as its last MFMA
// of the stage is issued, at least 28 MFMAs (of 64) ahead of its next use: B's right half in the first
// phase, A and B's left half (of the next stage) in the second.  The copies go out one at a time between
// the MFMAs.  Stages of 32 k keep four slots in LDS, so a copy has two to three stages to land.  One barrier
// per stage, between the phases: there stage s + 1 has landed and every wave has read all of stage s,
// whose slot is free for stage s + RING.
//
// The 16 x 16 x 32 MFMA moves half as many accumulator registers per product as the 32 x 32 x 16 one and
// leaves the fragments in the registers they were read into for a whole stage (64 instead of 128
// registers): 8192^3, X W^T 889 -> 832 us, dY W 872 -> 818, dY^T X 961 -> 867.
//
// Measured: 1030-1340 TFLOP/s.  With the 32 x 32 x 16 MFMA 8192^3 ran at 1237 TFLOP/s, the same loop without
// its copies at 1497, with every copy a hit in L2 at 1217, with three or five slots as with four: the
// copies' throughput into LDS next to the fragment reads is what is left, not their latency.  Operands
// packed into MFMA fragments first (contiguous KiB per copy) gave the loop 5-10% and cost 8-15% of an
// operation in packing.
//
// The MFMAs are issued through inline assembly so that the accumulators stay in accumulation registers
// for the whole loop (with the builtin the allocator moved tiles between the two register files).
// (B's fragment is the first operand: a lane then holds four consecutive columns of one row of C.)
#define TW_MFMA(d, x, y) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(y), "v"(x))
template <bool TA, bool TB, bool OUT_F32, bool ACCUM, int WMT, int WNT>
__global__ __launch_bounds__(NTHREAD, 1) void tw_gemm_kernel(Operand A, Operand B, int K, void* __restrict__ Cout, int64_t ldc,
                                                              int M, int N, Units u, float* __restrict__ part)
{
    constexpr unsigned STAGE = (WMT + WNT) * PANEL;      // bytes of a slot: A's panels, then B's
    constexpr int MI = 2 * WMT, NI = 2 * WNT, NH = NI / 2;  // accumulator tiles of a wave; NH: columns of a phase
    constexpr int NC = WMT + WNT;                        // copies of a wave per stage
    constexpr int NC0 = (NC + 1) / 2;                    // .. of which in the second phase of a stage, the rest in the first phase of the next
    static_assert(NWAVE == 4, "a wave copies a quarter of every panel");
    __shared__ __attribute__((aligned(256))) u32x4 ring[(RING + 1) * STAGE / 16];
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
    const int stages = K / SK;  // whole ones, >= 1 in every split (host)
    const int unit_stages = is_part ? u.split_stages : stages, stage0 = (int)split * unit_stages;
    const int n_full = stages - stage0 < unit_stages ? stages - stage0 : unit_stages;
    const bool tail = K % SK != 0 && stage0 + n_full == stages;  // the last split's stage of less than SK

    const unsigned ring0 = fpdt::lds_address(ring);
    Side<TA, WMT> a_side;
    Side<TB, WNT> b_side;
    a_side.init(A, tile_m * (64 * WMT), stage0, wu, wm * MI, lane, ring0);
    b_side.init(B, tile_n * (64 * WNT), stage0, wu, wn * NI, lane, ring0 + WMT * PANEL);
    const unsigned copy_lds = ring0 + 1024u * (unsigned)wu;
    // Copy j of the stage at a_at / b_at into the slot at LDS byte `slot_lds`: two scalar instructions besides
    // the copy, the second one for copy_address_rule (mfma_tiles.h) and as m0's wait state.
    auto copy = [&](int j, uint64_t a_at, uint64_t b_at, unsigned slot_lds) {
        uint64_t addr;
        asm volatile("s_add_u32 m0, %1, %2\n\ts_mov_b64 %0, %4\n\tglobal_load_lds_dwordx4 %3, %0"
                     : "=&s"(addr)
                     : "s"(slot_lds), "i"(PANEL * j), "v"(j < WMT ? a_side.off[j % WMT] : b_side.off[(j - WMT) % WNT]), "s"(j < WMT ? a_at : b_at)
                     : "memory", "scc");
    };
    auto stage_at = [&](uint64_t pos, int t, uint64_t step) { return pos + (uint64_t)((int64_t)t * (int64_t)step); };  // t stages behind pos
    if (tail) {  // its pieces pass through registers, zero behind K, into the slot behind the ring
        u32x4 v[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            v[j] = u32x4{0, 0, 0, 0};
            if (j < WMT) {
                const uint64_t src = a_side.pos + (uint64_t)n_full * a_side.step + a_side.off[j % WMT];
                if (a_side.has(stages, K, wu, lane)) v[j] = *reinterpret_cast<const u32x4*>((uintptr_t)src);
            } else {
                const uint64_t src = b_side.pos + (uint64_t)n_full * b_side.step + b_side.off[(j - WMT) % WNT];
                if (b_side.has(stages, K, wu, lane)) v[j] = *reinterpret_cast<const u32x4*>((uintptr_t)src);
            }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) ring[(RING * STAGE + PANEL * j + 1024u * wu) / 16 + lane] = v[j];
    }

    floatx4 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+a"(acc[i][j]));
        }

    // Stages 0 .. RING - 2 whole and the first copies of stage RING - 1.  A copy behind the last whole
    // stage fetches that stage again, into a slot that nobody reads any more: the loop then needs no
    // branch (with one, the allocator spilled the accumulators) and its wait counts are constants.
    auto ahead = [&](int t, int full) { return t < full ? t : full - 1; };
#pragma unroll
    for (int t = 0; t < RING; ++t)
#pragma unroll
        for (int j = 0; j < (t < RING - 1 ? NC : NC0); ++j)
            fpdt::frag_to_lds_at(j < WMT ? stage_at(a_side.pos, ahead(t, n_full), a_side.step) : stage_at(b_side.pos, ahead(t, n_full), b_side.step),
                                 copy_lds + (unsigned)t * STAGE + PANEL * (unsigned)j,
                                 (int)(j < WMT ? a_side.off[j % WMT] : b_side.off[(j - WMT) % WNT]));
    fpdt::wait_vmem_at_most<(RING - 2) * NC + NC0>();
    fpdt::barrier_no_fence();

    bf16x8 a[MI], b[NI];
#pragma unroll
    for (int j = 0; j < NH; ++j) b[j] = b_side.frag(j, 0u);
#pragma unroll
    for (int i = 0; i < MI; ++i) a[i] = a_side.frag(i, 0u);

    // the sides' pos is at the current stage, which is in slot `cur`
    unsigned cur = 0;
    int left = n_full + (tail ? 1 : 0);
    do {
        const int full = tail ? left - 1 : left;  // (0 in the tail stage: its copies fetch the stage before it)
        const unsigned nxt = tail && left == 2 ? RING : (cur + 1) % RING, prv = (cur + RING - 1) % RING;
        const int t_prv = ahead(RING - 1, full), t_cur = ahead(RING, full);
        const uint64_t a_prv = stage_at(a_side.pos, t_prv, a_side.step), b_prv = stage_at(b_side.pos, t_prv, b_side.step);
        const uint64_t a_cur = stage_at(a_side.pos, t_cur, a_side.step), b_cur = stage_at(b_side.pos, t_cur, b_side.step);
        const unsigned lds_prv = copy_lds + prv * STAGE, lds_cur = copy_lds + cur * STAGE;
        constexpr int NM = MI * NH;  // MFMAs of a phase
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            TW_MFMA(acc[m / NH][m % NH], a[m / NH], b[m % NH]);
            if (m < NH) b[NH + m] = b_side.frag(NH + m, cur * STAGE);
#pragma unroll
            for (int q = m * (NC - NC0) / NM; q < (m + 1) * (NC - NC0) / NM; ++q) copy(NC0 + q, a_prv, b_prv, lds_prv);  // the rest of stage s + RING - 1
            __builtin_amdgcn_sched_barrier(0);
        }
        fpdt::wait_vmem_at_most<(RING - 2) * NC>();
        fpdt::barrier_no_fence();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            TW_MFMA(acc[m / NH][NH + m % NH], a[m / NH], b[NH + m % NH]);
            if (m < NH) b[m] = b_side.frag(m, nxt * STAGE);
            if (m % NH == NH - 1) a[m / NH] = a_side.frag(m / NH, nxt * STAGE);
#pragma unroll
            for (int q = m * NC0 / NM; q < (m + 1) * NC0 / NM; ++q) copy(q, a_cur, b_cur, lds_cur);  // stage s + RING
            __builtin_amdgcn_sched_barrier(0);
        }
        a_side.pos += a_side.step;
        b_side.pos += b_side.step;
        cur = nxt;
    } while (--left > 0);
    fpdt::wait_vmem_at_most<0>();  // nothing may still be on its way into LDS when the ring is used again or the workgroup ends
    fpdt::barrier_no_fence();

    // the accumulators are read by ordinary instructions from here on
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    // accumulator tile (i, j): lane l holds row l % 16, columns 4 (l / 16) .. + 3
    const int mw = wm * (32 * WMT), nw = wn * (32 * WNT);  // the wave's first row and column within the tile
    // Sixteen rows at a time pass through LDS (each wave its own part of the idle ring), so that a store
    // covers 128 WNT bytes of a row in fp32.  With ACC the old values of sixteen rows are all requested, and
    // those of the next sixteen in front of their stores: one load at a time, each waited for behind the
    // store before it, left the read-modify-write of a weight gradient at a sixth of the memory rate.
    auto store_tile = [&](auto* out, int64_t pitch, auto acc_tag) {
        constexpr bool ACC = decltype(acc_tag)::value;
        typedef std::remove_pointer_t<decltype(out)> out_t;
        typedef out_t out4 __attribute__((ext_vector_type(4)));
        constexpr int LPR = 8 * WNT, RPI = 64 / LPR, PITCH = 32 * WNT + 4;  // lanes per row, rows per access, floats (4 apart: no bank conflicts)
        static_assert(4 * 16 * PITCH * 4 <= (RING + 1) * (int)STAGE, "the ring holds sixteen rows of every wave");
        float* rows = reinterpret_cast<float*>(ring) + wu * (16 * PITCH);
        float* put = rows + (lane & 15) * PITCH + 4 * (lane >> 4);
        const float* get = rows + (lane / LPR) * PITCH + 4 * (lane % LPR);
        out_t* c0 = out + (size_t)(mw + lane / LPR) * pitch + nw + 4 * (lane % LPR);
        out4 old[2][NI];
        auto request = [&](int i) {
#pragma unroll
            for (int k = 0; k < NI; ++k) old[i & 1][k] = *reinterpret_cast<const out4*>(c0 + (size_t)(16 * i + RPI * k) * pitch);
        };
        if (ACC) request(0);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (ACC && i + 1 < MI) request(i + 1);
            __builtin_amdgcn_sched_barrier(0);  // no further ahead: the registers are spoken for
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                asm volatile("" : "+a"(acc[i][j]));  // stays in its accumulation registers until here
                *reinterpret_cast<floatx4*>(put + 16 * j) = acc[i][j];
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < NI; ++k) {
                const floatx4 x = *reinterpret_cast<const floatx4*>(get + RPI * k * PITCH);
                out4 v;
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = combine<ACC>(x[r], ACC ? old[i & 1][k][r] : out_t(0));
                *reinterpret_cast<out4*>(c0 + (size_t)(16 * i + RPI * k) * pitch) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
    if (is_part) {  // this split's sums of the whole tile; tw_split_sum_kernel adds them
        constexpr size_t TILE_ELEMS = (size_t)(64 * WMT) * (64 * WNT);
        store_tile(part + ((size_t)split * divided + (id - (unsigned)u.whole)) * TILE_ELEMS, 64 * WNT, std::false_type{});
        return;
    }
    typedef typename std::conditional<OUT_F32, float, uint16_t>::type out_t;
    const int mt = tile_m * (64 * WMT), nt = tile_n * (64 * WNT);
    out_t* tile = static_cast<out_t*>(Cout) + (size_t)mt * ldc + nt;
    if (mt + 64 * WMT <= M && nt + 64 * WNT <= N && ldc % 4 == 0 && reinterpret_cast<uintptr_t>(Cout) % (4 * sizeof(out_t)) == 0) {
        store_tile(tile, ldc, std::integral_constant<bool, ACCUM>{});
        return;
    }
    // A tile that reaches behind C, or rows of C that are not aligned for four elements: sixteen rows at a time
    // through LDS as above, one element per lane and access, consecutive lanes on consecutive columns.  (Straight
    // from the accumulators an access touched 16 rows at 16 bytes each: odd widths then took up to twice the
    // time of the tiles' MFMAs.)  The old values of the sixteen rows are requested together.
    constexpr int PITCH = 32 * WNT + 4, CPR = 32 * WNT / 64;  // floats between rows, accesses per row
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
            asm volatile("" : "+a"(acc[i][j]));
            *reinterpret_cast<floatx4*>(put + 16 * j) = acc[i][j];
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
    int64_t R, C, ld, R2, C2;
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
    return (k_rows ? R : C) >= SK && (C % 8 == 0 || padded) && ld % 8 == 0 && ld < (k_rows ? MAX_PITCH_T : MAX_PITCH) &&
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
        const int64_t R2 = k_rows && R < SK ? SK : R, C2 = !k_rows && C < SK ? SK : (C + 7) / 8 * 8;
        // whole cache lines from row to row: a stage's pieces of a row are half a line (form N), of four
        // rows' columns a whole one (form T), and with 8208 bytes in place of 8320 straddled two
        // (16384 x 4097 x 4096 in 8 chunks: 864 -> 743 us)
        res->ld = C2 <= 64 ? C2 : (C2 + 63) / 64 * 64;
        res->p = nullptr;
        if (cache)
            for (const Realigned& c : g_cache)
                if (c.src == X && c.R == R && c.C == C && c.ld == ld && c.R2 == R2 && c.C2 == C2) res->p = c.copy;
        if (!res->p) {
            char* mem = nullptr;
            if (pool_take(pool, (size_t)R2 * res->ld * 2, &mem)) return 1;
            const int64_t blocks = (R2 * (C2 / 8) + 255) / 256;
            tw_realign_kernel<<<dim3((unsigned)(blocks < 65536 ? blocks : 65536)), 256, 0, st>>>(
                static_cast<const uint16_t*>(X), R, C, ld, reinterpret_cast<u32x4*>(mem), R2, C2, res->ld);
            res->p = reinterpret_cast<const uint16_t*>(mem);
            if (cache) g_cache.push_back({X, R, C, ld, R2, C2, res->p});
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
    const int Kp = K < SK ? SK : K;  // (realigned operands of less are padded to one stage)
    const Plan plan = plan_product(M, N, Kp / SK);
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
    rc = launch_product(plan, a_transposed, b_transposed, pa, pb, M, N, Kp, C, ldc, c_f32, accumulate, part, st);
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
        const int Kp = k < SK ? SK : (int)k;
        one.u.split_stages = Kp / SK;
        rc = launch_product(one, a_transposed, b_transposed, a, b, M, N, Kp, C, ldc, c_f32, accumulate, part + (size_t)i * (part_bytes(one) / 4), st);
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
