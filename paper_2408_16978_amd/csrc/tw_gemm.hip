// Dense bf16 products of the token-wise chunked operations (Sec. 4.1, 5.4: the per-chunk QKV
// projection, the feed-forward block and the output projection of the loss are plain GEMMs over
// one chunk of tokens at a time) on v_mfma_f32_32x32x16_bf16, with the operand machinery of the
// attention kernels: operands re-laid once into 1 KiB MFMA fragments, a four-slot LDS ring
// filled by direct global -> LDS copies three stages ahead, four waves (one per SIMD) per
// output tile of up to 256 x 256.
//
//   C[M,N] (+)= sum_k Aop[m,k] * Bop[n,k]          fp32 accumulation, C bf16 or fp32
//
// Every product of the library is of this form once each operand is read either as stored
// (row = row, k = column) or transposed (row = column, k = row); the pack kernel does both, pads
// rows to a multiple of 256 and k to a multiple of the stage depth with zeros, so the product kernel has no
// edge cases on its reads; its stores are bounds-checked.
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

// ---- pack -------------------------------------------------------------------------------
// X [R, C] bf16 row-major, leading dimension ld.  transposed = 0: fragment rows are rows of X,
// the contraction runs over its columns; 1: fragment rows are columns of X, the contraction
// runs over its rows.  out[rb][kt][lane][8]: lane (r = lane % 32, h = lane / 32) of fragment
// (rb, kt) holds element (row 32 rb + r, k = 16 kt + 8 h + e), e = 0..7; zero outside X.
// One workgroup: 32 fragment rows x 64 contraction indices (four fragments).
__global__ __launch_bounds__(256) void tw_pack_kernel(const uint16_t* __restrict__ X, int64_t R, int64_t C, int64_t ld,
                                                      int transposed, u32x4* __restrict__ out, int KT, int KC)
{
    __shared__ uint16_t tile[32][64 + 2];
    const int tid = threadIdx.x;
    const unsigned rb = blockIdx.x / (unsigned)KC, kc = blockIdx.x % (unsigned)KC;  // KC = chunks of 64 along k
    const int64_t row0 = (int64_t)rb * 32, k0 = (int64_t)kc * 64;
    // 256 threads x 8 consecutive elements of X = the 32 x 64 tile; 16-byte loads where the row
    // allows it (8 elements inside the matrix, 16-byte aligned), element by element at the edges
    auto load8 = [&](int64_t gr, int64_t gc0, uint16_t (&e)[8]) {
        const uint16_t* src = X + gr * ld + gc0;
        if (gr < R && gc0 + 8 <= C && (reinterpret_cast<uintptr_t>(src) & 15) == 0) {
            const uint4 v = *reinterpret_cast<const uint4*>(src);
            e[0] = (uint16_t)v.x; e[1] = (uint16_t)(v.x >> 16); e[2] = (uint16_t)v.y; e[3] = (uint16_t)(v.y >> 16);
            e[4] = (uint16_t)v.z; e[5] = (uint16_t)(v.z >> 16); e[6] = (uint16_t)v.w; e[7] = (uint16_t)(v.w >> 16);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = (gr < R && gc0 + j < C) ? src[j] : (uint16_t)0;
        }
    };
    uint16_t e8[8];
    if (!transposed) {
        const int r = tid >> 3, k = (tid & 7) * 8;  // row r of the tile, contraction indices k .. k + 7
        load8(row0 + r, k0 + k, e8);
#pragma unroll
        for (int j = 0; j < 8; ++j) tile[r][k + j] = e8[j];
    } else {
        const int k = tid >> 2, r = (tid & 3) * 8;  // row k0 + k of X, its columns row0 + r .. + 7
        load8(k0 + k, row0 + r, e8);
#pragma unroll
        for (int j = 0; j < 8; ++j) tile[r + j][k] = e8[j];
    }
    __syncthreads();
    const int t = tid >> 6, lane = tid & 63;
    const int kt = (int)kc * 4 + t;
    if (kt < KT) {
        const int r = lane & 31, h = lane >> 5;
        uint16_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = tile[r][16 * t + 8 * h + j];
        u32x4 v;
        v[0] = e[0] | ((unsigned)e[1] << 16);
        v[1] = e[2] | ((unsigned)e[3] << 16);
        v[2] = e[4] | ((unsigned)e[5] << 16);
        v[3] = e[6] | ((unsigned)e[7] << 16);
        out[((size_t)rb * KT + kt) * 64 + lane] = v;
    }
}

// ---- product ----------------------------------------------------------------------------
constexpr int NWAVE = 4, NTHREAD = NWAVE * 64;
constexpr int TILE = 256;  // packed operands are padded to this many rows
constexpr int SKT = 2;     // k-steps of 16 per LDS stage
constexpr int RING = 4;    // LDS slots of one stage each

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t b) { return __uint_as_float((unsigned)b << 16); }

// Af, Bf: packed operands (row blocks padded to the tile, KT a multiple of SKT).  C [M, N] row-major,
// leading dimension ldc elements.  A workgroup of four waves, one per SIMD, computes a (64 WMT) x
// (64 WNT) tile over the k-steps of its split; wave (w / 2, w % 2) owns WMT x WNT accumulator tiles.
//
// What bounds it: LDS traffic next to the MFMAs.  A wave reads WMT + WNT fragments (1 KiB) per
// WMT * WNT MFMAs, so the 128 x 128 elements of a wave at WMT = WNT = 4 need 0.5 fragments per MFMA;
// eight waves of 128 x 64 need 0.75, and with the copies' writes LDS was then as busy as the MFMA
// pipes.  The 256 accumulator registers leave room for one wave per SIMD, so nothing but this wave's
// own instruction order hides a latency: fragments are read one k-step ahead into a second register
// set, one read behind every MFMA, and the copies go out one at a time between the MFMAs.
// Stages of 32 k keep four slots in LDS, so a copy has two to three stages to land.  One barrier per
// stage, in its middle: there stage s + 1 has landed and every wave has read all of stage s, whose
// slot is free for stage s + RING.  Eight waves and 64-deep stages before, here (4096 rows): 14336 -> 4096
// 409 -> 386 us, 1060 x 4096 x 128256 2128 -> 968 us (there the k splits), with fp32 accumulation into
// 14336 x 4096 580 -> 478 us (there the epilogue below).
// The MFMAs are issued through inline assembly so that the accumulators stay in accumulation registers
// for the whole loop (with the builtin the allocator moved tiles between the two register files).
#define TW_MFMA(d, x, y) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(x), "v"(y))
template <bool OUT_F32, bool ACCUM, int WMT, int WNT>
__global__ __launch_bounds__(NTHREAD, 1) void tw_gemm_kernel(const u32x4* __restrict__ Af, const u32x4* __restrict__ Bf,
                                                              int KT, void* __restrict__ Cout, int64_t ldc, int M, int N,
                                                              int tiles_n, int tiles_total, int splits, int split_stages)
{
    constexpr int NA = 2 * WMT, NB = 2 * WNT;            // row blocks of a stage
    constexpr int STAGE_U4 = (NA + NB) * SKT * 64;
    constexpr int NC = WMT + WNT;                        // copies of a wave per stage
    constexpr int NC0 = (NC + 1) / 2;                    // .. of which in the first of the two k-steps that issue them
    static_assert(SKT == 2 && NWAVE == 4, "a wave copies one k-step of every second block");
    __shared__ u32x4 ring[RING * STAGE_U4];
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
    const int stage0 = (int)split * split_stages;
    const int n_stages = KT / SKT - stage0 < split_stages ? KT / SKT - stage0 : split_stages;  // >= 1 (host)

    // This wave copies k-step wu % 2 of the blocks wu / 2, wu / 2 + 2, .. of each operand.
    const uint64_t blk_bytes = (uint64_t)KT * 1024;
    const uint64_t first = (uint64_t)(wu >> 1) * blk_bytes + (uint64_t)(wu & 1) * 1024 + (uint64_t)stage0 * (SKT * 1024);
    uint64_t a_src = fpdt::uniform((uint64_t)(uintptr_t)Af + (uint64_t)tile_m * NA * blk_bytes + first);
    uint64_t b_src = fpdt::uniform((uint64_t)(uintptr_t)Bf + (uint64_t)tile_n * NB * blk_bytes + first);
    const unsigned ring_lds = fpdt::lds_address(ring) + 1024u * (unsigned)wu;  // block wu / 2, k-step wu % 2
    const int lane16 = 16 * lane;
    auto copy = [&](int j, uint64_t ahead, unsigned slot) {  // copy j of the stage `ahead` bytes behind a_src / b_src
        const uint64_t src = (j < WMT ? a_src : b_src) + (uint64_t)(2 * (j < WMT ? j : j - WMT)) * blk_bytes + ahead;
        const unsigned blk = (unsigned)(j < WMT ? 2 * j : NA + 2 * (j - WMT));
        fpdt::frag_to_lds_at(src, ring_lds + slot * (STAGE_U4 * 16u) + blk * (SKT * 1024u), lane16);
    };

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

    // stages 0 .. RING - 2 whole and the first copies of stage RING - 1.  A copy behind the last stage
    // fetches that stage again, into a slot that nobody reads any more: the loop then needs no branch
    // (with one, the allocator spilled the accumulators) and its wait counts are constants.
    auto ahead = [&](int t, int left) { return (uint64_t)(unsigned)(t < left ? t : left - 1) * (SKT * 1024); };
#pragma unroll
    for (int t = 0; t < RING; ++t)
#pragma unroll
        for (int j = 0; j < (t < RING - 1 ? NC : NC0); ++j) copy(j, ahead(t, n_stages), (unsigned)t);
    fpdt::wait_vmem_at_most<(RING - 2) * NC + NC0>();
    fpdt::barrier_no_fence();

    bf16x8 a[2][WMT], b[2][WNT];
    const u32x4* mine = ring + lane;
    auto read = [&](int set, int i, const u32x4* slot) {  // fragment i of the set, b first: the order of use
        if (i < WNT) b[set][i] = fpdt::as_bf16x8(slot[((NA + wn * WNT + i) * SKT + set) * 64]);
        else a[set][i - WNT] = fpdt::as_bf16x8(slot[((wm * WMT + i - WNT) * SKT + set) * 64]);
    };
#pragma unroll
    for (int i = 0; i < NC; ++i) read(0, i, mine);

    // a_src / b_src point at the current stage, which is in slot `cur`
    unsigned cur = 0;
    int left = n_stages;
    do {
        const unsigned nxt = (cur + 1) % RING, prv = (cur + RING - 1) % RING;
        const u32x4* sl = mine + cur * STAGE_U4;
        const u32x4* nsl = mine + nxt * STAGE_U4;
        const uint64_t ahead_prv = ahead(RING - 1, left), ahead_cur = ahead(RING, left);
        // reads in the first half of a k-step (they are waited for at its end), copies all over it
        constexpr int NM = WMT * WNT, NH = NM / 2;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            TW_MFMA(acc[m / WNT][m % WNT], a[0][m / WNT], b[0][m % WNT]);
#pragma unroll
            for (int q = m * NC / NH; q < (m + 1) * NC / NH && q < NC; ++q) read(1, q, sl);
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
            for (int q = m * NC / NH; q < (m + 1) * NC / NH && q < NC; ++q) read(0, q, nsl);
#pragma unroll
            for (int q = m * NC0 / NM; q < (m + 1) * NC0 / NM; ++q) copy(q, ahead_cur, cur);  // stage s + RING
            __builtin_amdgcn_sched_barrier(0);
        }
        a_src += SKT * 1024;
        b_src += SKT * 1024;
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

// ---- host side: packed-operand scratch and the per-call cache of packed weights --------------
struct Pool {
    char* base = nullptr;
    size_t cap = 0, off = 0;
    std::vector<void*> retired;  // outgrown buffers: work already enqueued may still read them
};
struct Packed {
    const void* src;
    int64_t R, C, ld;
    int transposed;
    const u32x4* frags;
    int RB, KT;
};
Pool g_pool[64];
std::vector<Packed> g_cache;  // weights packed during the current library call
std::mutex g_mu;

size_t packed_bytes(int64_t rows, int64_t k, int tile, int* RB, int* KT)
{
    *RB = (int)((rows + tile - 1) / tile * (tile / 32));
    *KT = (int)((k + 16 * SKT - 1) / (16 * SKT) * SKT);
    return (size_t)*RB * *KT * 1024;
}

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

int pack_operand(Pool& pool, const void* X, int64_t R, int64_t C, int64_t ld, int transposed, int tile,
                 bool cache, hipStream_t st, Packed* res)
{
    if (cache)
        for (const Packed& c : g_cache)
            if (c.src == X && c.R == R && c.C == C && c.ld == ld && c.transposed == transposed) {
                *res = c;
                return 0;
            }
    Packed p{X, R, C, ld, transposed, nullptr, 0, 0};
    const int64_t rows = transposed ? C : R, k = transposed ? R : C;
    const size_t bytes = packed_bytes(rows, k, tile, &p.RB, &p.KT);
    char* mem = nullptr;
    if (pool_take(pool, bytes, &mem)) return 1;
    p.frags = reinterpret_cast<const u32x4*>(mem);
    const int KC = (p.KT + 3) / 4;
    if ((long long)p.RB * KC > (1ll << 30)) return 2;
    tw_pack_kernel<<<dim3((unsigned)(p.RB * KC)), 256, 0, st>>>(static_cast<const uint16_t*>(X), R, C, ld, transposed,
                                                               reinterpret_cast<u32x4*>(mem), p.KT, KC);
    if (cache) g_cache.push_back(p);
    *res = p;
    return 0;
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
    const Plan plan = plan_product(M, N, (int)(((int64_t)K + 16 * SKT - 1) / (16 * SKT)));
    const int tile_rows = 64 * plan.wmt, tile_cols = 64 * plan.wnt;
    const int tiles_n = (N + tile_cols - 1) / tile_cols, tiles_m = (M + tile_rows - 1) / tile_rows;
    const long long total = (long long)tiles_m * tiles_n;
    if (total * plan.splits > (1ll << 30)) return 2;
    // Aop[m,k]: A stored [M,K] (as is) or [K,M] (transposed); Bop[n,k]: B stored [N,K] or [K,N]
    Packed pa, pb;
    int rc = pack_operand(pool, B, b_transposed ? K : N, b_transposed ? N : K, ldb, b_transposed, TILE, cache_b, st, &pb);
    if (rc) return rc;
    const size_t mark = pool.off;  // what follows is scratch of this product only
    rc = pack_operand(pool, A, a_transposed ? K : M, a_transposed ? M : K, lda, a_transposed, tile_rows, false, st, &pa);
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
    const int KT = pa.KT;  // = pb.KT: both contract over K
#define TW_LAUNCH_TILE(F32, ACC, WM, WN)                                                                            \
    tw_gemm_kernel<F32, ACC, WM, WN><<<grid, NTHREAD, 0, st>>>(pa.frags, pb.frags, KT, out, out_ld, M, N, tiles_n,   \
                                                               (int)total, plan.splits, plan.split_stages)
#define TW_LAUNCH(F32, ACC)                                             \
    do {                                                                \
        if (plan.wnt == 2) TW_LAUNCH_TILE(F32, ACC, 2, 2);              \
        else if (plan.wmt == 4) TW_LAUNCH_TILE(F32, ACC, 4, 4);         \
        else if (plan.wmt == 3) TW_LAUNCH_TILE(F32, ACC, 3, 4);         \
        else if (plan.wmt == 2) TW_LAUNCH_TILE(F32, ACC, 2, 4);         \
        else TW_LAUNCH_TILE(F32, ACC, 1, 4);                            \
    } while (0)
    if (plan.splits > 1 || (c_f32 && !accumulate)) TW_LAUNCH(true, false);
    else if (c_f32) TW_LAUNCH(true, true);
    else if (accumulate) TW_LAUNCH(false, true);
    else TW_LAUNCH(false, false);
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
    // The next product's packs run after this launch on the same stream, so this product's scratch
    // is free again: everything it took, or everything behind a weight that stays cached.  (Not if
    // the pool was replaced by a larger one on the way: then nothing is given back until the next
    // library call.)
    if (pool.base == base0) pool.off = cache_b ? mark : off0;
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace fpdt_tw
