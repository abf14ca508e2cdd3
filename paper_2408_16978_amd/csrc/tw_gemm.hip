// Dense bf16 products of the token-wise chunked operations (Sec. 4.1, 5.4: the per-chunk QKV
// projection, the feed-forward block and the output projection of the loss are plain GEMMs over
// one chunk of tokens at a time) on v_mfma_f32_32x32x16_bf16: a four-slot LDS ring filled by direct
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

#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>
#include <vector>

#include "mfma_tiles.h"
#include "tw_gemm.h"

namespace fpdt_tw {

using fpdt::bf16x8;
using fpdt::floatx16;
using fpdt::u32x4;

namespace {

// ---- realign ----------------------------------------------------------------------------
// The product kernel copies 16-byte pieces of its operands' rows and needs at least one whole stage of
// k.  An operand that does not offer that (a width that is not a multiple of 8, a base that is not
// 16-byte aligned, k < 32) is copied once into out [R2, C2], zero behind X [R, C].
__global__ __launch_bounds__(256) void tw_realign_kernel(const uint16_t* __restrict__ X, int64_t R, int64_t C, int64_t ld,
                                                         u32x4* __restrict__ out, int64_t R2, int64_t C2)
{
    const int64_t pieces = C2 / 8, n = R2 * pieces;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t r = i / pieces, c = i % pieces * 8;
        unsigned e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = r < R && c + j < C ? X[r * ld + c + j] : 0u;
        out[i] = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
}

// ---- product ----------------------------------------------------------------------------
constexpr int NWAVE = 4, NTHREAD = NWAVE * 64;
constexpr int SK = 32;        // k per LDS stage: two MFMA k-steps
constexpr int RING = 4;       // LDS slots of one stage each; one more holds a last stage of less than SK
constexpr unsigned PANEL = 4096;  // bytes of a panel: 64 rows of one operand x SK

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((unsigned)b << 16); }

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
//   Form T: panel row k (128 bytes, 64 columns) holds its two 64-byte halves at half ^ (k / 2) % 2: the four
//           k x 32 columns that half a wave's transposing read covers lie in different 64-byte columns of
//           256 bytes.
template <bool T, int NP>
struct Side {
    uint64_t pos;        // scalar: the current stage
    uint64_t step;       // bytes from a stage to the next
    uint64_t rel[NP];    // scalar: panel j's quarter
    unsigned off[NP];    // this lane's piece of it
    unsigned rd[2];      // LDS bytes within a stage: form N k-step 0 / 1, form T even / odd fragments

    __device__ __forceinline__ void init(const Operand& x, int row0, int stage0, int w, int wave_frag0, int lane, unsigned lds0)
    {
        const uint64_t pitch = (uint64_t)x.ld * 2;
        const int limit = x.rows - row0;  // >= 1
        if (T) {
            step = SK * pitch;
            pos = (uint64_t)(uintptr_t)(x.p + row0) + (uint64_t)stage0 * step + (uint64_t)(8 * w) * pitch;
            const int k = lane >> 3, half = ((lane >> 2) & 1) ^ ((k >> 1) & 1);
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                const int c = 64 * j + 32 * half + 8 * (lane & 3);
                rel[j] = 0;
                off[j] = (unsigned)k * (unsigned)pitch + 2u * (unsigned)(c < limit - 8 ? c : limit - 8);
            }
            const int grp = lane >> 4, e = (lane & 15) >> 2, x4 = lane & 3;
            const unsigned lane_part = 128u * (unsigned)(8 * (grp >> 1) + e) + 32u * (unsigned)(grp & 1) + 8u * (unsigned)x4;
#pragma unroll
            for (int par = 0; par < 2; ++par) {
                const int f = wave_frag0 + par;
                rd[par] = lds0 + PANEL * (unsigned)(f >> 1) + 64u * (unsigned)((f & 1) ^ (e >> 1)) + lane_part;
            }
        } else {
            step = SK * 2;
            pos = (uint64_t)(uintptr_t)x.p + (uint64_t)row0 * pitch + (uint64_t)stage0 * step;
            const int r = lane >> 2, q = (lane & 3) ^ ((r >> 1) & 3) ^ ((r >> 3) & 1);
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                // rows behind the operand are read as its last row: their products are not stored
                const int first = 64 * j + 16 * w < limit ? 64 * j + 16 * w : limit - 1;
                const int mine = 64 * j + 16 * w + r < limit ? 64 * j + 16 * w + r : limit - 1;
                rel[j] = (uint64_t)first * pitch;
                off[j] = (unsigned)(mine - first) * (unsigned)pitch + 16u * (unsigned)q;
            }
            const int fr = lane & 15, swz = ((fr >> 1) & 3) ^ ((fr >> 3) & 1);
            rd[0] = lds0 + 64u * (unsigned)(32 * wave_frag0 + (lane & 31)) + 16u * (unsigned)((lane >> 5) ^ swz);
            rd[1] = rd[0] ^ 32u;
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
    // fragment i of the wave, k-step t, of the stage at LDS byte `slot`
    __device__ __forceinline__ bf16x8 frag(int i, int t, unsigned slot) const
    {
        if (T) {
            typedef short short4v __attribute__((ext_vector_type(4)));
            typedef short short8v __attribute__((ext_vector_type(8)));
            typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
            const unsigned at = rd[i & 1] + slot + PANEL * (unsigned)(i >> 1) + 2048u * (unsigned)t;
            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)at);
            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(at + 512u));
            const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        }
        typedef __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
        return fpdt::as_bf16x8(*(lds_u32x4_ptr)(uintptr_t)(rd[t] + slot + 2048u * (unsigned)i));
    }
};

// C [M, N] row-major, leading dimension ldc elements.  A workgroup of four waves, one per SIMD, computes a
// (64 WMT) x (64 WNT) tile over the stages of its split; wave (w / 2, w % 2) owns WMT x WNT accumulator
// tiles of 32 x 32.
//
// What bounds it: LDS traffic next to the MFMAs.  A wave reads WMT + WNT fragments (1 KiB) per
// WMT * WNT MFMAs, so the 128 x 128 elements of a wave at WMT = WNT = 4 need 0.5 fragments per MFMA;
// eight waves of 128 x 64 need 0.75, and with the copies' writes LDS was then as busy as the MFMA
// pipes.  The 256 accumulator registers leave room for one wave per SIMD, so nothing but this wave's
// own instruction order hides a latency: fragments are read one k-step ahead into a second register
// set, one read behind every MFMA, and the copies go out one at a time between the MFMAs.
// Stages of 32 k keep four slots in LDS, so a copy has two to three stages to land.  One barrier per
// stage, in its middle: there stage s + 1 has landed and every wave has read all of stage s, whose
// slot is free for stage s + RING.
//
// Measured: 1030-1270 TFLOP/s (8192^3 in the three forms: 1240, 1267, 1136).  The same loop without its
// copies reaches 1300-1500, with every copy a hit in L2 1060-1220, with three or five slots the same as
// with four: the copies' throughput into LDS next to the fragment reads is what is left, not their
// latency.  Operands packed into MFMA fragments first (contiguous KiB per copy) gave the loop 5-10% and
// cost 8-15% of an operation in packing.
//
// The MFMAs are issued through inline assembly so that the accumulators stay in accumulation registers
// for the whole loop (with the builtin the allocator moved tiles between the two register files).
#define TW_MFMA(d, x, y) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(x), "v"(y))
template <bool TA, bool TB, bool OUT_F32, bool ACCUM, int WMT, int WNT>
__global__ __launch_bounds__(NTHREAD, 1) void tw_gemm_kernel(Operand A, Operand B, int K, void* __restrict__ Cout, int64_t ldc,
                                                              int M, int N, int tiles_n, int tiles_total, int splits, int split_stages)
{
    constexpr unsigned STAGE = (WMT + WNT) * PANEL;      // bytes of a slot: A's panels, then B's
    constexpr int NC = WMT + WNT;                        // copies of a wave per stage
    constexpr int NC0 = (NC + 1) / 2;                    // .. of which in the first of the two k-steps that issue them
    static_assert(NWAVE == 4, "a wave copies a quarter of every panel");
    __shared__ __attribute__((aligned(256))) u32x4 ring[(RING + 1) * STAGE / 16];
    // Consecutive workgroup ids land on different XCDs (each with its own L2): give every XCD a
    // contiguous run of tiles, so that the tiles that share an operand row share an L2.
    const unsigned work_total = (unsigned)tiles_total * (unsigned)splits;
    const unsigned per_xcd = (work_total + 7) / 8;
    const unsigned wid = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
    if (blockIdx.x / 8 >= per_xcd || wid >= work_total) return;  // whole workgroup, before any barrier
    const unsigned split = wid / (unsigned)tiles_total, id = wid % (unsigned)tiles_total;
    // Within a run the tiles go in groups of four tile rows, row index fastest: the 32 workgroups
    // that an XCD runs at a time then cover about 4 x 8 tiles and share 4 + 8 operand slices in its
    // L2 instead of 1 + 32.
    constexpr unsigned GROUP_M = 4;
    const unsigned tiles_m = (unsigned)tiles_total / (unsigned)tiles_n;
    const unsigned grp = id / (GROUP_M * (unsigned)tiles_n), in_grp = id % (GROUP_M * (unsigned)tiles_n);
    const unsigned rows_in_grp = tiles_m - grp * GROUP_M < GROUP_M ? tiles_m - grp * GROUP_M : GROUP_M;
    const int tile_m = (int)(grp * GROUP_M + in_grp % rows_in_grp), tile_n = (int)(in_grp / rows_in_grp);

    const int lane = threadIdx.x & 63;
    const int wu = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wu >> 1, wn = wu & 1;
    const int stages = K / SK;  // whole ones, >= 1 in every split (host)
    const int stage0 = (int)split * split_stages;
    const int n_full = stages - stage0 < split_stages ? stages - stage0 : split_stages;
    const bool tail = K % SK != 0 && stage0 + n_full == stages;  // the last split's stage of less than SK

    const unsigned ring0 = fpdt::lds_address(ring);
    Side<TA, WMT> a_side;
    Side<TB, WNT> b_side;
    a_side.init(A, tile_m * (64 * WMT), stage0, wu, wm * WMT, lane, ring0);
    b_side.init(B, tile_n * (64 * WNT), stage0, wu, wn * WNT, lane, ring0 + WMT * PANEL);
    const unsigned copy_lds = ring0 + 1024u * (unsigned)wu;
    // copy j of the stage `t` stages behind the current one
    auto copy = [&](int j, int t, unsigned slot) {
        const unsigned dst = copy_lds + slot * STAGE + PANEL * (unsigned)j;
        if (j < WMT) fpdt::frag_to_lds_at(a_side.pos + a_side.rel[j % WMT] + (uint64_t)((int64_t)t * (int64_t)a_side.step), dst, (int)a_side.off[j % WMT]);
        else fpdt::frag_to_lds_at(b_side.pos + b_side.rel[(j - WMT) % WNT] + (uint64_t)((int64_t)t * (int64_t)b_side.step), dst, (int)b_side.off[(j - WMT) % WNT]);
    };
    if (tail) {  // its pieces pass through registers, zero behind K, into the slot behind the ring
        u32x4 v[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            v[j] = u32x4{0, 0, 0, 0};
            if (j < WMT) {
                const uint64_t src = a_side.pos + a_side.rel[j % WMT] + (uint64_t)n_full * a_side.step + a_side.off[j % WMT];
                if (a_side.has(stages, K, wu, lane)) v[j] = *reinterpret_cast<const u32x4*>((uintptr_t)src);
            } else {
                const uint64_t src = b_side.pos + b_side.rel[(j - WMT) % WNT] + (uint64_t)n_full * b_side.step + b_side.off[(j - WMT) % WNT];
                if (b_side.has(stages, K, wu, lane)) v[j] = *reinterpret_cast<const u32x4*>((uintptr_t)src);
            }
        }
#pragma unroll
        for (int j = 0; j < NC; ++j) ring[(RING * STAGE + PANEL * j + 1024u * wu) / 16 + lane] = v[j];
    }

    floatx16 acc[WMT][WNT];
#pragma unroll
    for (int i = 0; i < WMT; ++i)
#pragma unroll
        for (int j = 0; j < WNT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < WMT; ++i)
#pragma unroll
        for (int j = 0; j < WNT; ++j) asm volatile("" : "+a"(acc[i][j]));

    // Stages 0 .. RING - 2 whole and the first copies of stage RING - 1.  A copy behind the last whole
    // stage fetches that stage again, into a slot that nobody reads any more: the loop then needs no
    // branch (with one, the allocator spilled the accumulators) and its wait counts are constants.
    auto ahead = [&](int t, int full) { return t < full ? t : full - 1; };
#pragma unroll
    for (int t = 0; t < RING; ++t)
#pragma unroll
        for (int j = 0; j < (t < RING - 1 ? NC : NC0); ++j) copy(j, ahead(t, n_full), (unsigned)t);
    fpdt::wait_vmem_at_most<(RING - 2) * NC + NC0>();
    fpdt::barrier_no_fence();

    bf16x8 a[2][WMT], b[2][WNT];
    auto read = [&](int set, int i, unsigned slot) {  // fragment i of the set, b first: the order of use
        if (i < WNT) b[set][i % WNT] = b_side.frag(i, set, slot);
        else a[set][(i - WNT) % WMT] = a_side.frag(i - WNT, set, slot);
    };
#pragma unroll
    for (int i = 0; i < NC; ++i) read(0, i, 0u);

    // the sides' pos is at the current stage, which is in slot `cur`
    unsigned cur = 0;
    int left = n_full + (tail ? 1 : 0);
    do {
        const int full = tail ? left - 1 : left;  // (0 in the tail stage: its copies fetch the stage before it)
        const unsigned nxt = tail && left == 2 ? RING : (cur + 1) % RING, prv = (cur + RING - 1) % RING;
        const int ahead_prv = ahead(RING - 1, full), ahead_cur = ahead(RING, full);
        // reads in the first half of a k-step (they are waited for at its end), copies all over it
        constexpr int NM = WMT * WNT, NH = NM / 2;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            TW_MFMA(acc[m / WNT][m % WNT], a[0][m / WNT], b[0][m % WNT]);
#pragma unroll
            for (int q = m * NC / NH; q < (m + 1) * NC / NH && q < NC; ++q) read(1, q, cur * STAGE);
#pragma unroll
            for (int q = m * (NC - NC0) / NM; q < (m + 1) * (NC - NC0) / NM; ++q) copy(NC0 + q, ahead_prv, prv);  // the rest of stage s + RING - 1
            __builtin_amdgcn_sched_barrier(0);
        }
        fpdt::wait_vmem_at_most<(RING - 2) * NC>();
        fpdt::barrier_no_fence();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            TW_MFMA(acc[m / WNT][m % WNT], a[1][m / WNT], b[1][m % WNT]);
#pragma unroll
            for (int q = m * NC / NH; q < (m + 1) * NC / NH && q < NC; ++q) read(0, q, nxt * STAGE);
#pragma unroll
            for (int q = m * NC0 / NM; q < (m + 1) * NC0 / NM; ++q) copy(q, ahead_cur, cur);  // stage s + RING
            __builtin_amdgcn_sched_barrier(0);
        }
        a_side.pos += a_side.step;
        b_side.pos += b_side.step;
        cur = nxt;
    } while (--left > 0);
    fpdt::wait_vmem_at_most<0>();  // nothing may still be on its way into LDS when the workgroup ends

    // the accumulators are read by ordinary instructions from here on
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    // accumulator tile (i, j): lane l holds column l % 32, register r row 8 (r / 4) + 4 (l / 32) + r % 4.
    // With ACCUM the old values of two tiles are all requested, and those of the next two in front
    // of their stores: one load at a time, each waited for behind the store before it, left the
    // read-modify-write of a weight gradient at a sixth of the memory rate.
    const int col = lane & 31, half = lane >> 5;
    const int m0 = tile_m * (64 * WMT) + wm * (32 * WMT) + 4 * half, n0 = tile_n * (64 * WNT) + wn * (32 * WNT) + col;
    typedef typename std::conditional<OUT_F32, float, uint16_t>::type out_t;
    // (splits > 1: fp32, this split's sums)
    out_t* c0 = static_cast<out_t*>(Cout) + (size_t)split * (splits > 1 ? (size_t)M * N : 0) + (size_t)m0 * ldc + n0;
    auto epilogue = [&](auto inside_tag) {  // INSIDE: no element of the tile lies behind C
        constexpr bool INSIDE = decltype(inside_tag)::value;
        auto row = [&](int i, int r) { return 32 * i + 8 * (r >> 2) + (r & 3); };
        auto in = [&](int i, int j, int r) { return INSIDE || (m0 + row(i, r) < M && n0 + 32 * j < N); };
        constexpr int NU = WMT * WNT / 2;  // units of two tiles side by side
        out_t old[2][2][16];
        auto request = [&](int u) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = 2 * u / WNT, j = 2 * u % WNT + jj;
                    old[u & 1][jj][r] = 0;
                    if (in(i, j, r)) old[u & 1][jj][r] = c0[(size_t)row(i, r) * ldc + 32 * j];
                }
        };
        if (ACCUM) request(0);
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (ACCUM && u + 1 < NU) request(u + 1);
            __builtin_amdgcn_sched_barrier(0);  // no further ahead: the registers are spoken for
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int i = 2 * u / WNT, j = 2 * u % WNT + jj;
                    if (in(i, j, r)) {
                        const float v = acc[i][j][r];
                        if constexpr (OUT_F32) c0[(size_t)row(i, r) * ldc + 32 * j] = ACCUM ? old[u & 1][jj][r] + v : v;
                        else c0[(size_t)row(i, r) * ldc + 32 * j] = to_bf16(ACCUM ? from_bf16(old[u & 1][jj][r]) + v : v);
                    }
                }
        }
    };
    if ((tile_m + 1) * (64 * WMT) <= M && (tile_n + 1) * (64 * WNT) <= N) epilogue(std::true_type{});
    else epilogue(std::false_type{});
}

// C (+)= the splits' sums, part [splits][M * N] fp32; V consecutive elements of C per thread (V divides N,
// ldc and the alignment).  Memory-bound: (splits + 1) passes over C.
template <bool OUT_F32, bool ACCUM, int V>
__global__ __launch_bounds__(256) void tw_split_sum_kernel(const float* __restrict__ part, int splits, int64_t MN, int N,
                                                            void* __restrict__ Cout, int64_t ldc)
{
    typedef float fvec __attribute__((ext_vector_type(V)));
    typedef uint16_t hvec __attribute__((ext_vector_type(V)));
    const int64_t at = ((int64_t)blockIdx.x * 256 + threadIdx.x) * V;
    if (at >= MN) return;
    fvec v = *reinterpret_cast<const fvec*>(part + at);
    for (int s = 1; s < splits; ++s) v += *reinterpret_cast<const fvec*>(part + s * MN + at);
    const int64_t c = at / N * ldc + at % N;
    if (OUT_F32) {
        fvec* o = reinterpret_cast<fvec*>(static_cast<float*>(Cout) + c);
        *o = ACCUM ? *o + v : v;
    } else {
        hvec* o = reinterpret_cast<hvec*>(static_cast<uint16_t*>(Cout) + c);
        hvec h;
        if (ACCUM) h = *o;
#pragma unroll
        for (int e = 0; e < V; ++e) h[e] = to_bf16(ACCUM ? from_bf16(h[e]) + v[e] : v[e]);
        *o = h;
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

// Output tile (64 wmt x 64 wnt) and number of k splits of a product: the cheapest in units of the
// core clock, from
//   stage   the MFMAs of a wave (32 clocks each) or, on the small tiles, the fragments that pass
//           through LDS (reads and copies, 128 bytes per clock), and about 100 for the barrier
//   tile    a fixed part (first operands, epilogue), rounds of 256 tiles (512 where two fit a CU)
//   splits  one more launch and (splits + 1) passes over the fp32 sums at about 4.5 bytes per ns
struct Plan { int wmt, wnt, splits, split_stages; };
Plan plan_product(int64_t M, int64_t N, int stages)
{
    static const int shapes[][2] = {{4, 4}, {3, 4}, {2, 4}, {1, 4}, {2, 2}};
    Plan best = {4, 4, 1, stages};
    double best_cost = 0.0;
    for (const auto& sh : shapes) {
        const int wm = sh[0], wn = sh[1];
        const double lds = 96.0 * (wm + wn), mfma = 64.0 * wm * wn;
        const double stage = (mfma > lds ? mfma : lds) + 100.0;
        const double slots = wm * wn <= 4 && wn == 2 ? 512.0 : 256.0, share = slots / 256.0;
        const double tiles = (double)((M + 64 * wm - 1) / (64 * wm)) * (double)((N + 64 * wn - 1) / (64 * wn));
        for (int sp = 1; sp <= 16; ++sp) {
            const int per = (stages + sp - 1) / sp;
            if (sp > 1 && (per < 8 || (int64_t)(sp - 1) * per >= stages)) continue;
            if (sp > 1 && (double)M * (double)N * sp > 1.0e8) break;  // the sums would not stay near the chip
            double cost = std::ceil(tiles * sp / slots) * share * (per * stage + 1200.0 + 10.0 * wm * wn * 16);
            if (sp > 1) cost += 9000.0 + (sp + 1) * 4.0 * (double)M * (double)N / 2250.0;
            if (best_cost == 0.0 || cost < 0.98 * best_cost) {
                best = {wm, wn, sp, per};
                best_cost = cost;
            }
        }
    }
    return best;
}

int pool_take(Pool& p, size_t bytes, char** out)
{
    bytes = (bytes + 255) & ~(size_t)255;
    if (p.off + bytes > p.cap) {
        // grow: a new buffer; the old one stays alive (kernels in flight may read it) until exit
        size_t want = p.cap ? p.cap * 2 : (size_t)256 << 20;
        while (want < bytes) want *= 2;
        void* nb = nullptr;
        if (hipMalloc(&nb, want) != hipSuccess) {
            (void)hipGetLastError();
            return 1;
        }
        if (p.base) p.retired.push_back(p.base);
        p.base = static_cast<char*>(nb);
        p.cap = want;
        p.off = 0;
        g_cache.clear();  // cached fragments lived in the old buffer
    }
    *out = p.base + p.off;
    p.off += bytes;
    return 0;
}

// X [R, C], leading dimension ld, as the product kernel can read it: in place, or copied.  `k_rows`: the
// contraction runs over the rows of X.  `padded`: rows are followed by zeros up to a multiple of 8.
int take_operand(Pool& pool, const void* X, int64_t R, int64_t C, int64_t ld, bool k_rows, bool padded, bool cache, hipStream_t st, Operand* res)
{
    const int64_t K = k_rows ? R : C;
    res->rows = (int)(k_rows ? (C + 7) / 8 * 8 : R);
    if (K >= SK && (C % 8 == 0 || padded) && ld % 8 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0) {
        res->p = static_cast<const uint16_t*>(X);
        res->ld = ld;
    } else {
        const int64_t R2 = k_rows && R < SK ? SK : R, C2 = !k_rows && C < SK ? SK : (C + 7) / 8 * 8;
        res->ld = C2;
        res->p = nullptr;
        if (cache)
            for (const Realigned& c : g_cache)
                if (c.src == X && c.R == R && c.C == C && c.ld == ld && c.R2 == R2 && c.C2 == C2) res->p = c.copy;
        if (!res->p) {
            char* mem = nullptr;
            if (pool_take(pool, (size_t)R2 * C2 * 2, &mem)) return 1;
            const int64_t blocks = (R2 * (C2 / 8) + 255) / 256;
            tw_realign_kernel<<<dim3((unsigned)(blocks < 65536 ? blocks : 65536)), 256, 0, st>>>(
                static_cast<const uint16_t*>(X), R, C, ld, reinterpret_cast<u32x4*>(mem), R2, C2);
            res->p = reinterpret_cast<const uint16_t*>(mem);
            if (cache) g_cache.push_back({X, R, C, ld, R2, C2, res->p});
        }
    }
    // a lane's offset from its quarter panel (15 rows of form N, 7 of form T) is kept in 32 bits
    return res->ld >= (int64_t)1 << 27 ? 2 : 0;
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

void* scratch(size_t bytes)
{
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
    char* mem = nullptr;
    return pool_take(g_pool[dev], bytes, &mem) ? nullptr : mem;
}

int gemm(int a_transposed, int b_transposed, int M, int N, int K, const void* A, int64_t lda, const void* B,
         int64_t ldb, void* C, int64_t ldc, bool c_f32, bool accumulate, bool cache_b, hipStream_t st)
{
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1;
    Pool& pool = g_pool[dev];
    if (M <= 0 || N <= 0 || K <= 0) return 2;
    const char* base0 = pool.base;
    const size_t off0 = pool.off;
    const int Kp = K < SK ? SK : K;  // (realigned operands of less are padded to one stage)
    const Plan plan = plan_product(M, N, Kp / SK);
    const int tile_rows = 64 * plan.wmt, tile_cols = 64 * plan.wnt;
    const int tiles_n = (N + tile_cols - 1) / tile_cols, tiles_m = (M + tile_rows - 1) / tile_rows;
    const long long total = (long long)tiles_m * tiles_n;
    if (total * plan.splits > (1ll << 30)) return 2;
    // Aop[m,k]: A stored [M,K] (as is) or [K,M] (transposed); Bop[n,k]: B stored [N,K] or [K,N]
    Operand pa, pb;
    int rc = take_operand(pool, B, b_transposed ? K : N, b_transposed ? N : K, ldb, b_transposed, false, cache_b, st, &pb);
    if (rc) return rc;
    const size_t mark = pool.off;  // what follows is scratch of this product only
    rc = take_operand(pool, A, a_transposed ? K : M, a_transposed ? M : K, lda, a_transposed, lda > (a_transposed ? M : K), false, st, &pa);
    if (rc) return rc;
    void* out = C;
    int64_t out_ld = ldc;
    if (plan.splits > 1) {
        char* mem = nullptr;
        if (pool_take(pool, (size_t)plan.splits * M * N * 4, &mem)) return 1;
        out = mem;
        out_ld = N;
    }
    const unsigned grid = (unsigned)((total * plan.splits + 7) / 8 * 8);
#define TW_LAUNCH_TILE(TA, TB, F32, ACC, WM, WN)                                                                     \
    tw_gemm_kernel<TA, TB, F32, ACC, WM, WN><<<grid, NTHREAD, 0, st>>>(pa, pb, Kp, out, out_ld, M, N, tiles_n,        \
                                                                       (int)total, plan.splits, plan.split_stages)
#define TW_LAUNCH(TA, TB, F32, ACC)                                             \
    do {                                                                        \
        if (plan.wnt == 2) TW_LAUNCH_TILE(TA, TB, F32, ACC, 2, 2);              \
        else if (plan.wmt == 4) TW_LAUNCH_TILE(TA, TB, F32, ACC, 4, 4);         \
        else if (plan.wmt == 3) TW_LAUNCH_TILE(TA, TB, F32, ACC, 3, 4);         \
        else if (plan.wmt == 2) TW_LAUNCH_TILE(TA, TB, F32, ACC, 2, 4);         \
        else TW_LAUNCH_TILE(TA, TB, F32, ACC, 1, 4);                            \
    } while (0)
    const bool f32 = c_f32 || plan.splits > 1, add = accumulate && plan.splits == 1;
    // the forms and outputs that the library's operations use
    if (!a_transposed && !b_transposed && !add) {
        if (f32) TW_LAUNCH(false, false, true, false);
        else TW_LAUNCH(false, false, false, false);
    } else if (!a_transposed && b_transposed && !(f32 && add)) {
        if (f32) TW_LAUNCH(false, true, true, false);
        else if (add) TW_LAUNCH(false, true, false, true);
        else TW_LAUNCH(false, true, false, false);
    } else if (a_transposed && b_transposed && f32) {
        if (add) TW_LAUNCH(true, true, true, true);
        else TW_LAUNCH(true, true, true, false);
    } else {
        return 2;
    }
#undef TW_LAUNCH
#undef TW_LAUNCH_TILE
    if (plan.splits > 1) {
        const int64_t MN = (int64_t)M * N;
        const bool v4 = N % 4 == 0 && ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % (c_f32 ? 16 : 8) == 0;
        const unsigned blocks = (unsigned)((MN / (v4 ? 4 : 1) + 255) / 256);
        const float* part = static_cast<const float*>(out);
#define TW_SUM(F32, ACC)                                                                                  \
    do {                                                                                                  \
        if (v4) tw_split_sum_kernel<F32, ACC, 4><<<blocks, 256, 0, st>>>(part, plan.splits, MN, N, C, ldc); \
        else tw_split_sum_kernel<F32, ACC, 1><<<blocks, 256, 0, st>>>(part, plan.splits, MN, N, C, ldc);    \
    } while (0)
        if (c_f32 && accumulate) TW_SUM(true, true);
        else if (c_f32) TW_SUM(true, false);
        else if (accumulate) TW_SUM(false, true);
        else TW_SUM(false, false);
#undef TW_SUM
    }
    // The next product's copies run after this launch on the same stream, so this product's scratch
    // is free again: everything it took, or everything behind a weight that stays cached.  (Not if
    // the pool was replaced by a larger one on the way: then nothing is given back until the next
    // library call.)
    if (pool.base == base0) pool.off = cache_b ? mark : off0;
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace fpdt_tw
