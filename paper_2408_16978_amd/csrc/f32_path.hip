// fp32 accuracy path, partial-result merge and fill kernels.
//
// The fp32 kernels compute the chunked attention on v_mfma_f32_16x16x4_f32 (fp32 operands, fp32
// accumulation) in the formulation of the bf16 kernels: forward and dQ hold S^T = K Q^T (a lane owns one
// query), dK/dV hold S = Q K^T (a lane owns one key), and the register-resident score tile is the next
// product's operand.  Their tensors are small (the accuracy configuration has 1K tokens), so what bounds
// them is the chain of one row tile and the number of launches: tiles have 16 rows (of 32 rows there are
// 64 at 1K tokens and two heads, a quarter of the compute units), the eight waves of a workgroup share a
// tile, each walking every eighth 16-row block of the other side, and their results meet in LDS; a call
// without FPDT_PAIRWISE is one forward and one backward launch.  At 1024 tokens, 2 heads, D = 64, chunks of 256, forward
// and backward: one wave per row with scalar dot products, pair by pair, 1799 us; 32-row tiles 110 us; 16-row tiles
// whose operands are fetched where they are used, rows and again columns, and whose addresses are vector arithmetic
// (64-bit divisions among it), 64 us; this 48 us (twelve or sixteen waves: no faster).  Errors against fp64 are below those
// of the scalar kernels in O, dQ, dK and dV (2.5e-7 .. 7.0e-7 against 3.3e-7 .. 9.7e-7 over four shapes).
#include "fpdt_internal.h"
#include "mfma_tiles.h"

namespace fpdt {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// acc[16x16] += A[16x4] B[4x16]: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and of the result
// column l % 16, rows 4 (l / 16) + r
__device__ __forceinline__ floatx4 mfma_f32(float a, float b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int NW = 8;    // waves of a workgroup
constexpr int TR = 16;   // rows of a tile
constexpr int BR = 16;   // rows of a block of the other side

// Row operand of a product contracted over the channels: lane (row = lane % 16, g = lane / 16) holds
// channels 16 j + 4 g + 0..3, j = 0 .. D/16 - 1, of its row.  (Any order of the channels does, as both
// operands use the same.)
template <int D>
struct Rows {
    f32x4 v[D / 16];
    __device__ __forceinline__ void load(const float* row, int g)
    {
#pragma unroll
        for (int j = 0; j < D / 16; ++j) v[j] = *reinterpret_cast<const f32x4*>(row + 16 * j + 4 * g);
    }
};
template <int D>
__device__ __forceinline__ floatx4 dot_rows(const Rows<D>& a, const Rows<D>& b)
{
    floatx4 s = {};
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) s = mfma_f32(a.v[j][c], b.v[j][c], s);
    return s;
}

// A wave's own part of LDS: the rows of `PLACES` blocks, for the products contracted over them, and a score tile.  (Rows 4 floats
// apart from a multiple of the banks: what a read takes, sixteen elements of every fourth row, lies in different ones.)
template <int D, int PLACES>
struct Shelf {
    static constexpr int PITCH = D + 4, ROWS = TR * PITCH, FLOATS = PLACES * ROWS + TR * TR;
    float* p;
    int lane;
    // Rows x into place `at`, zeros for elements that are not finite; are there any?
    __device__ __forceinline__ bool put(int at, const Rows<D>& x) const
    {
        float z = 0.f;
#pragma unroll
        for (int j = 0; j < D / 16; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) z = fmaf(x.v[j][c], 0.f, z);  // not a number if one is not finite
        const bool odd = __any(!(z == 0.f));
        f32x4* to = reinterpret_cast<f32x4*>(p + at * ROWS + (lane & 15) * PITCH + 4 * (lane >> 4));
#pragma unroll
        for (int j = 0; j < D / 16; ++j) to[4 * j] = x.v[j];
        if (__builtin_expect(odd, 0)) {
#pragma unroll
            for (int j = 0; j < D / 16; ++j) {
                f32x4 v = x.v[j];
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = fabsf(v[c]) < INFINITY ? v[c] : 0.f;
                to[4 * j] = v;
            }
        }
        __builtin_amdgcn_wave_barrier();
        return odd;
    }
    // Column operand: element 16 db + lane % 16 of row 4 (lane / 16) + r
    __device__ __forceinline__ float get(int at, int db, int r) const { return p[at * ROWS + (4 * (lane >> 4) + r) * PITCH + 16 * db + (lane & 15)]; }
    __device__ __forceinline__ float* tile() const { return p + PLACES * ROWS; }
};

// acc^T [D x 16] += X^T [D x 16 rows] T [16 rows x 16 columns]: `t` is a score tile in accumulator layout
// (this lane: column lane % 16, rows 4 (lane / 16) + r), the rows of X are in place `at` of the shelf.  `keep` has
// bit r set where t[r] counts; where it does not, t[r] is 0, but the row of X may hold infinities or NaN (a
// later key of this query), which 0 times it must not let through: those elements (`odd`: there are some) stay
// out of the product and are added one by one where they count.
template <int D, int PLACES>
__device__ __forceinline__ void add_rows(floatx4 (&acc)[D / 16], const floatx4& t, unsigned keep, const Shelf<D, PLACES>& shelf, int at, bool odd,
                                         const float* X, size_t pitch, int n_rows, int lane)
{
    const int g = lane >> 4, col = lane & 15;
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[db] = mfma_f32(shelf.get(at, db, r), t[r], acc[db]);
    if (__builtin_expect(odd, 0)) {
        // t by row through LDS; a NaN pattern that no arithmetic produces marks what does not count
        float* park = shelf.tile();
#pragma unroll
        for (int r = 0; r < 4; ++r) park[(4 * g + r) * 16 + col] = (keep >> r) & 1 ? t[r] : __uint_as_float(0xffffdeadu);
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int row = 0; row < n_rows; ++row) {
            const float p = park[row * 16 + col];
            const bool on = __float_as_uint(p) != 0xffffdeadu;
#pragma unroll
            for (int db = 0; db < D / 16; ++db) {
                const f32x4 v = *reinterpret_cast<const f32x4*>(X + (size_t)row * pitch + 16 * db + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (on && !(fabsf(v[e]) < INFINITY)) acc[db][e] += p * v[e];
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Sum over the waves of a workgroup of acc^T [D x 16] (and of more_acc^T), and the result to out(0, d, column) (out(1, d, column)) for
// every element (17 floats per channel: the final reads, channel fastest, then fall into different banks)
template <int D, bool MORE, typename F>
__device__ __forceinline__ void sum_waves(const floatx4 (&acc)[D / 16], const floatx4 (&more_acc)[D / 16], float* lds, F out)
{
    constexpr int ALL = D * 17, WAVES = NW * ALL;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    __syncthreads();
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            lds[w * ALL + (16 * db + 4 * g + r) * 17 + col] = acc[db][r];
            if (MORE) lds[WAVES + w * ALL + (16 * db + 4 * g + r) * 17 + col] = more_acc[db][r];
        }
    __syncthreads();
    // channel fastest over the threads: rows of the result are written in whole lines
    for (int e = threadIdx.x; e < D * TR; e += NW * 64) {
        const int d = e % D, c = e / D;
        float v = lds[d * 17 + c], x = MORE ? lds[WAVES + d * 17 + c] : 0.f;
#pragma unroll
        for (int i = 1; i < NW; ++i) {
            v += lds[i * ALL + d * 17 + c];
            if (MORE) x += lds[WAVES + i * ALL + d * 17 + c];
        }
        out(0, d, c, v);
        if (MORE) out(1, d, c, x);
    }
}

__device__ __forceinline__ float max_over_rows(float v)  // over the four lanes of a column
{
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float sum_over_rows(float v)
{
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// Workgroup = one 16-query tile of one head; wave w folds key blocks w, w + 8, .. into its own (max, sum,
// un-normalised output), wave 0 starting from the carried state; they are merged at the end.
//
// At D = 64 and 80 two workgroups fit a compute unit, where one runs its products under the other's exponentials (D = 80, 32 / 8
// heads, 1K tokens: one 117 us, two 90).  Tiles start with the longest walks; between 257 and 512 of them, which then all start at
// once, the shortest follow on the 256 longest, so that what shares a compute unit is about the same everywhere (D = 80, 4 heads, 2K
// tokens: one at a time 51 us, two in order 63, this 47; D = 64: in order 52, this 39).
template <int D>
__global__ __launch_bounds__(64 * NW, D == 128 ? 2 : 4) void f32_fwd_kernel(F32FwdArgs a)
{
    constexpr int DB = D / 16;
    typedef Shelf<D, 1> MyShelf;
    static_assert(MyShelf::FLOATS >= D * 17, "sum_waves uses the same memory");
    __shared__ __attribute__((aligned(16))) float lds[NW * MyShelf::FLOATS];
    __shared__ float ml[NW][2][TR];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
    const int n_tiles = (int)((a.n_q + TR - 1) / TR);
    const unsigned turn = D < 128 && gridDim.x <= 512 && blockIdx.x >= 256 ? gridDim.x - 1 - (blockIdx.x - 256) : blockIdx.x;
    const int head = turn % (unsigned)a.Hq, tile = n_tiles - 1 - (int)(turn / (unsigned)a.Hq);  // longest first
    const int kvh = head / (a.Hq / a.Hkv);
    const int64_t row0 = (int64_t)tile * TR;
    const int rows = (int)(a.n_q - row0 < TR ? a.n_q - row0 : TR), my_row = col < rows ? col : rows - 1;
    const size_t q_pitch = (size_t)a.Hq * D, k_pitch = (size_t)a.Hkv * D;
    const int64_t qpos = a.q_pos0 + row0 + my_row;
    Rows<D> q;
    q.load(a.Q + (size_t)(row0 + my_row) * q_pitch + (size_t)head * D, g);

    float m = -INFINITY, l = 0.f;
    floatx4 acc[DB] = {};
    if (w == 0 && !(a.flags & SWEEP_INIT) && col < rows) {
        const size_t at = (size_t)(row0 + col) * a.Hq + head;
        m = a.st_ml[2 * at];
        l = g == 0 ? a.st_ml[2 * at + 1] : 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[db][r] = a.st_acc[at * D + 16 * db + 4 * g + r];
    }
    int64_t need = a.q_pos0 + row0 + rows - a.k_pos0;  // keys at positions <= the last query's
    if (need > a.n_k) need = a.n_k;
    // Rows are fetched once, 16 bytes per lane, the next block's as soon as this one's have been consumed, so that they
    // arrive under its products; the products contracted over rows take their operand from the wave's shelf in LDS.
    // (Fetched again as columns, 4 bytes per lane and access, where they are used: forward 22.6 us, backward 40.)
    auto keys_at = [&](int64_t j) { return (int)(a.n_k - j < BR ? a.n_k - j : BR); };
    auto row_at = [&](int64_t j) { return (j + (col < keys_at(j) ? col : keys_at(j) - 1)) * k_pitch + (size_t)kvh * D; };
    const MyShelf shelf = {lds + w * MyShelf::FLOATS, lane};
    Rows<D> k, v;
    if (BR * w < need) {
        k.load(a.K + row_at(BR * w), g);
        v.load(a.V + row_at(BR * w), g);
    }
#pragma unroll 1
    for (int64_t j0 = BR * w; j0 < need; j0 += BR * NW) {
        const int keys = keys_at(j0);
        floatx4 s = dot_rows<D>(k, q);
        const bool odd = shelf.put(0, v);
        if (j0 + BR * NW < need) {
            k.load(a.K + row_at(j0 + BR * NW), g);
            v.load(a.V + row_at(j0 + BR * NW), g);
        }
        unsigned keep = 0;
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int key = 4 * g + r;
            const bool on = key < keys && a.k_pos0 + j0 + key <= qpos;
            keep |= (unsigned)on << r;
            s[r] = on ? a.scale * s[r] : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        // Where no row of the tile has a new maximum nothing is exchanged or rescaled.  (A reference that moves only when a
        // score exceeds it by 2 or 8 is no faster and adds 4% to the error of the LSE.)
        // (every score of this wave so far may be -infinity, masked or overflowed: then 0 takes the maximum's
        // place, whatever was added is 0, and so stays what the next finite score rescales)
        if (__any(mx > m)) {
            const float m_new = fmaxf(m, max_over_rows(mx));
            const float alpha = expf(m - (m_new > -INFINITY ? m_new : 0.f));
            l *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[db][r] *= alpha;
            m = m_new;
        }
        const float m_ref = m > -INFINITY ? m : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = (keep >> r) & 1 ? expf(s[r] - m_ref) : 0.f;
            l += s[r];
        }
        add_rows(acc, s, keep, shelf, 0, odd, a.V + j0 * k_pitch + (size_t)kvh * D, k_pitch, keys, lane);
    }
    l = sum_over_rows(l);
    if (g == 0) {
        ml[w][0][col] = m;
        ml[w][1][col] = l;
    }
    __syncthreads();
    float m_all = ml[0][0][col], l_all = 0.f;
#pragma unroll
    for (int i = 1; i < NW; ++i) m_all = fmaxf(m_all, ml[i][0][col]);
#pragma unroll
    for (int i = 0; i < NW; ++i) l_all += ml[i][1][col] == 0.f ? 0.f : ml[i][1][col] * expf(ml[i][0][col] - m_all);
    const bool empty = l == 0.f;  // a wave without keys of this row adds nothing (its maximum is -infinity)
    const float mine = expf(m - m_all);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[db][r] = empty ? 0.f : acc[db][r] * mine;
    const bool final = a.flags & SWEEP_FINAL;
    __syncthreads();
    if (w == 0 && g == 0) {
        if (col < rows) {
            if (final) {
                a.LSE[(size_t)head * a.lse_stride + row0 + col] = m_all + logf(l_all);
            } else {
                const size_t at = (size_t)(row0 + col) * a.Hq + head;
                a.st_ml[2 * at] = m_all;
                a.st_ml[2 * at + 1] = l_all;
            }
        }
        ml[0][1][col] = final ? 1.f / l_all : 1.f;
    }
    sum_waves<D, false>(acc, acc, lds, [&](int, int d, int c, float v) {
        if (c < rows) (final ? a.O : a.st_acc)[((size_t)(row0 + c) * a.Hq + head) * D + d] = v * ml[0][1][c];
    });
}

// What the two workgroups of a tile hand over to each other.  They may run on different XCDs, whose L2 caches are not coherent: every access to
// these floats has the device's scope, which takes it past those caches to the memory that all of them see, and there are no others
// (the memory is private to this class; a plain load or store of it could be stale, or be seen late).  What orders them is
// not the language's (all are relaxed) but the chip's: a store of that scope has reached that memory when vmcnt counts it down, each
// wave waits for its own in front of the barrier, and only behind the barrier is the arrival counted, in the same memory; who
// finds the other's arrival there loads behind a second barrier.  (Ordered by the language, with a fence, each workgroup writes back an XCD's whole L2:
// 179 us instead of 29 at 1K tokens.)
class SharedSums {
    float* const part_;
    unsigned* const arrived_;

public:
    __device__ SharedSums(const F32BwdArgs& a, unsigned tile, int floats) : part_(a.part + (size_t)tile * floats), arrived_(a.arrived + tile) {}
    __device__ void store(int at, float v) const { __hip_atomic_store(part_ + at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ float load(int at) const { return __hip_atomic_load(part_ + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    // All stores of this workgroup are done; are the other's too?  (By the whole workgroup.)
    __device__ bool both_stored() const
    {
        __shared__ unsigned before;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) before = __hip_atomic_fetch_add(arrived_, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        return before != 0;
    }
};

// One launch for both sides: the first tiles are of 16 queries (dQ), the others of 16 keys (dK, dV:
// all query heads of the group).  Waves share the walk of a tile as in the forward.
//
// SPLIT (f32_bwd_split): two workgroups share a tile, each wave taking every 16th block.  Both store their sums; the one that arrives second
// adds the two (always in the same order) and writes the result.  Nobody waits.  Tiles start with the longest walks, of both
// kinds, so the second halves go in reverse: a compute unit then has a long and a short tile.  (Two workgroups on a compute unit at
// D = 64 take 25 registers of a loop to scratch memory: 28.9 us instead of 31.6 at 1K tokens, 2 / 2 heads, where one a tile takes 29.3, and
// 18.7 instead of 15.6 at 512.)
template <int D, bool SPLIT>
__global__ __launch_bounds__(64 * NW) void f32_bwd_kernel(F32BwdArgs a, unsigned dq_blocks, unsigned tiles)
{
    constexpr int DB = D / 16, STRIDE = SPLIT ? 2 * NW : NW;  // of the blocks of a walk that a wave takes
    __shared__ __attribute__((aligned(16))) float lds[NW * Shelf<D, 2>::FLOATS];
    const unsigned half = SPLIT && blockIdx.x >= tiles ? 1 : 0, tile_id = half ? 2 * tiles - 1 - blockIdx.x : blockIdx.x;
    const SharedSums sums(a, tile_id, 2 * (2 * TR * D));  // two halves of up to two results
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
    const int group = a.Hq / a.Hkv, first = w + NW * (int)half;
    const size_t q_pitch = (size_t)a.Hq * D, k_pitch = (size_t)a.Hkv * D;
    const Shelf<D, 2> shelf = {lds + w * Shelf<D, 2>::FLOATS, lane};
    if (tile_id < dq_blocks) {
        const int n_tiles = (int)((a.n_q + TR - 1) / TR);
        const int head = tile_id % (unsigned)a.Hq, tile = n_tiles - 1 - (int)(tile_id / (unsigned)a.Hq);
        const int kvh = head / group;
        const int64_t row0 = (int64_t)tile * TR;
        const int rows = (int)(a.n_q - row0 < TR ? a.n_q - row0 : TR), mine = col < rows ? col : rows - 1;
        const int64_t qpos = a.q_pos0 + row0 + mine;
        Rows<D> q, go;
        q.load(a.Q + (row0 + mine) * q_pitch + (size_t)head * D, g);
        go.load(a.dO + (row0 + mine) * q_pitch + (size_t)head * D, g);
        const float lse = a.LSE[(size_t)head * a.row_stat_stride + row0 + mine];
        const float delta = a.Delta[(size_t)head * a.row_stat_stride + row0 + mine];
        floatx4 acc[DB] = {};
        int64_t need = a.q_pos0 + row0 + rows - a.k_pos0;
        if (need > a.n_k) need = a.n_k;
        auto keys_at = [&](int64_t j) { return (int)(a.n_k - j < BR ? a.n_k - j : BR); };
        auto row_at = [&](int64_t j) { return (j + (col < keys_at(j) ? col : keys_at(j) - 1)) * k_pitch + (size_t)kvh * D; };
        Rows<D> k, v;  // (as in the forward)
        if (BR * first < need) {
            k.load(a.K + row_at(BR * first), g);
            v.load(a.V + row_at(BR * first), g);
        }
#pragma unroll 1
        for (int64_t j0 = BR * first; j0 < need; j0 += BR * STRIDE) {
            const int keys = keys_at(j0);
            const size_t k0 = j0 * k_pitch + (size_t)kvh * D;
            floatx4 s = dot_rows<D>(k, q);
            const bool odd = shelf.put(0, k);
            const floatx4 dp = dot_rows<D>(v, go);
            if (j0 + BR * STRIDE < need) {
                k.load(a.K + row_at(j0 + BR * STRIDE), g);
                v.load(a.V + row_at(j0 + BR * STRIDE), g);
            }
            unsigned keep = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = 4 * g + r;
                const bool on = key < keys && a.k_pos0 + j0 + key <= qpos;
                keep |= (unsigned)on << r;
                s[r] = on ? expf(a.scale * s[r] - lse) * (dp[r] - delta) : 0.f;
            }
            add_rows(acc, s, keep, shelf, 0, odd, a.K + k0, k_pitch, keys, lane);
        }
        auto put = [&](int d, int c, float v) {
            if (c < rows) {
                float* o = a.dQ + (row0 + c) * q_pitch + (size_t)head * D + d;
                *o = (a.accumulate ? *o : 0.f) + a.scale * v;
            }
        };
        if constexpr (SPLIT) {
            sum_waves<D, false>(acc, acc, lds, [&](int, int d, int c, float v) { sums.store((int)half * TR * D + c * D + d, v); });
            if (!sums.both_stored()) return;
            for (int e = threadIdx.x; e < TR * D; e += NW * 64) put(e % D, e / D, sums.load(e) + sums.load(TR * D + e));
        } else {
            sum_waves<D, false>(acc, acc, lds, [&](int, int d, int c, float v) { put(d, c, v); });
        }
        return;
    }
    const unsigned blk = tile_id - dq_blocks;
    const int kvh = blk % (unsigned)a.Hkv;
    const int64_t key0 = (int64_t)(blk / (unsigned)a.Hkv) * TR;  // first keys first: theirs is the longest walk
    const int keys = (int)(a.n_k - key0 < TR ? a.n_k - key0 : TR), mine = col < keys ? col : keys - 1;
    const int64_t kpos = a.k_pos0 + key0 + mine;
    Rows<D> k, v;
    k.load(a.K + (key0 + mine) * k_pitch + (size_t)kvh * D, g);
    v.load(a.V + (key0 + mine) * k_pitch + (size_t)kvh * D, g);
    floatx4 dk[DB] = {}, dv[DB] = {};
    int64_t i_first = a.k_pos0 + key0 - a.q_pos0;  // first query row that attends the tile's first key
    if (i_first < 0) i_first = 0;
    const int64_t blocks = i_first < a.n_q ? (a.n_q - i_first + BR - 1) / BR : 0;
    // the tile's walk: sixteen query rows of a head after the other, every NW-th of them by this wave
    struct Step {
        int64_t block;
        int head;
        __device__ __forceinline__ void forward(int64_t n, int64_t blocks)  // (no division: a walk has few heads)
        {
            block += n;
            while (block >= blocks) {
                block -= blocks;
                ++head;
            }
        }
    };
    auto rows_at = [&](int64_t i) { return (int)(a.n_q - i < BR ? a.n_q - i : BR); };
    auto row_at = [&](const Step& t) {
        const int64_t i = i_first + t.block * BR;
        return (i + (col < rows_at(i) ? col : rows_at(i) - 1)) * q_pitch + (size_t)(kvh * group + t.head) * D;
    };
    Rows<D> xq, xo;  // (as in the forward)
    auto load_rows = [&](const Step& t) {
        xq.load(a.Q + row_at(t), g);
        xo.load(a.dO + row_at(t), g);
    };
    Step t = {0, 0};
    if (blocks > 0) t.forward(first, blocks);
    else t.head = group;
    if (t.head < group) load_rows(t);
#pragma unroll 1
    while (t.head < group) {
        const int head = kvh * group + t.head;
        const int64_t i0 = i_first + t.block * BR;
        const int rows = rows_at(i0);
        const size_t q0 = i0 * q_pitch + (size_t)head * D;
        const float* lse = a.LSE + (size_t)head * a.row_stat_stride + i0;
        const float* delta = a.Delta + (size_t)head * a.row_stat_stride + i0;
        float ls[4], de[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            ls[r] = lse[4 * g + r < rows ? 4 * g + r : 0];
            de[r] = delta[4 * g + r < rows ? 4 * g + r : 0];
        }
        floatx4 s = dot_rows<D>(xq, k);
        const bool odd_q = shelf.put(0, xq);
        floatx4 ds = dot_rows<D>(xo, v);
        const bool odd_o = shelf.put(1, xo);
        t.forward(STRIDE, blocks);
        if (t.head < group) load_rows(t);
        unsigned keep = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * g + r;
            const bool on = row < rows && kpos <= a.q_pos0 + i0 + row;
            keep |= (unsigned)on << r;
            s[r] = on ? expf(a.scale * s[r] - ls[r]) : 0.f;
            ds[r] = on ? s[r] * (ds[r] - de[r]) : 0.f;
        }
        add_rows(dv, s, keep, shelf, 1, odd_o, a.dO + q0, q_pitch, rows, lane);
        add_rows(dk, ds, keep, shelf, 0, odd_q, a.Q + q0, q_pitch, rows, lane);
    }
    auto put = [&](int n, int d, int c, float x) {
        if (c < keys) {
            float* o = (n ? a.dV : a.dK) + (key0 + c) * k_pitch + (size_t)kvh * D + d;
            *o = (a.accumulate ? *o : 0.f) + (n ? 1.f : a.scale) * x;
        }
    };
    static_assert(NW * Shelf<D, 2>::FLOATS >= 2 * NW * D * 17, "both sums at a time");
    if constexpr (SPLIT) {
        sum_waves<D, true>(dk, dv, lds, [&](int n, int d, int c, float v) { sums.store((2 * n + (int)half) * TR * D + c * D + d, v); });
        if (!sums.both_stored()) return;
        for (int e = threadIdx.x; e < TR * D; e += NW * 64)
            for (int n = 0; n < 2; ++n) put(n, e % D, e / D, sums.load(2 * n * TR * D + e) + sums.load((2 * n + 1) * TR * D + e));
    } else {
        sum_waves<D, true>(dk, dv, lds, put);
    }
}

__device__ __forceinline__ float load_elem(const float* p) { return *p; }
__device__ __forceinline__ float load_elem(const uint16_t* p) { return __uint_as_float(((unsigned)*p) << 16); }
__device__ __forceinline__ void store_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(uint16_t* p, float v)
{
    const __bf16 b = (__bf16)v;  // round to nearest even
    *p = __builtin_bit_cast(uint16_t, b);
}

// 16 lanes per (row, head).
template <typename T>
__global__ __launch_bounds__(256) void merge_kernel(const T* Oa, const float* La, const T* Ob,
                                                    const float* Lb, T* Oo, float* Lo, int64_t rows,
                                                    int Hq, int D)
{
    const int64_t pair = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const int sub = threadIdx.x & 15;
    if (pair >= rows * Hq) return;
    const int64_t row = pair / Hq;
    const int h = (int)(pair % Hq);
    const float la = La[(size_t)h * rows + row], lb = Lb[(size_t)h * rows + row];
    const float mx = fmaxf(la, lb);
    float lse = -INFINITY, wa = 0.f, wb = 0.f;
    if (mx > -INFINITY) {
        lse = mx + logf(expf(la - mx) + expf(lb - mx));
        wa = expf(la - lse);
        wb = expf(lb - lse);
    }
    for (int d = sub; d < D; d += 16) {
        const size_t o = (size_t)pair * D + d;
        const float xa = wa > 0.f ? load_elem(Oa + o) : 0.f;
        const float xb = wb > 0.f ? load_elem(Ob + o) : 0.f;
        store_elem(Oo + o, wa * xa + wb * xb);
    }
    if (sub == 0) Lo[(size_t)h * rows + row] = lse;
}

__global__ __launch_bounds__(256) void fill_kernel(uint4* p, size_t n16, unsigned char* tail, int ntail, unsigned word)
{
    const size_t i0 = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t step = (size_t)gridDim.x * 256;
    for (size_t i = i0; i < n16; i += step) p[i] = make_uint4(word, word, word, word);
    if (blockIdx.x == 0 && (int)threadIdx.x < ntail) tail[threadIdx.x] = (unsigned char)word;
}

}  // namespace

void launch_f32_fwd(const F32FwdArgs& a, hipStream_t st)
{
    const dim3 grid((unsigned)((a.n_q + TR - 1) / TR * a.Hq));
    if (a.D == 128) f32_fwd_kernel<128><<<grid, 64 * NW, 0, st>>>(a);
    else if (a.D == 80) f32_fwd_kernel<80><<<grid, 64 * NW, 0, st>>>(a);
    else f32_fwd_kernel<64><<<grid, 64 * NW, 0, st>>>(a);
}

void launch_f32_bwd(const F32BwdArgs& a, hipStream_t st)
{
    const unsigned dq = (unsigned)((a.n_q + TR - 1) / TR * a.Hq);
    const unsigned tiles = dq + (unsigned)((a.n_k + TR - 1) / TR * a.Hkv);
#define F32_BWD(D_)                                                                             \
    do {                                                                                        \
        if (a.part) f32_bwd_kernel<D_, true><<<2 * tiles, 64 * NW, 0, st>>>(a, dq, tiles);      \
        else f32_bwd_kernel<D_, false><<<tiles, 64 * NW, 0, st>>>(a, dq, tiles);                \
    } while (0)
    if (a.D == 128) F32_BWD(128);
    else if (a.D == 80) F32_BWD(80);
    else F32_BWD(64);
#undef F32_BWD
}

size_t f32_bwd_part_bytes(int64_t S, int Hq, int Hkv, int D) { return (size_t)f32_bwd_tiles(S, Hq, Hkv) * (4 * TR * (size_t)D) * sizeof(float); }

void launch_merge(const void* Oa, const float* La, const void* Ob, const float* Lb, void* Oo,
                  float* Lo, int64_t rows, int Hq, int D, int is_bf16, hipStream_t st)
{
    const int64_t pairs = rows * Hq;
    dim3 grid((unsigned)((pairs + 15) / 16));
    if (is_bf16)
        merge_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)Oa, La, (const uint16_t*)Ob, Lb,
                                                     (uint16_t*)Oo, Lo, rows, Hq, D);
    else
        merge_kernel<float><<<grid, 256, 0, st>>>((const float*)Oa, La, (const float*)Ob, Lb,
                                                  (float*)Oo, Lo, rows, Hq, D);
}

void launch_zero(void* p, size_t bytes, hipStream_t st) { launch_fill_bytes(p, bytes, 0x00, st); }

void launch_fill_bytes(void* p, size_t bytes, unsigned char byte, hipStream_t st)
{
    if (bytes == 0) return;
    const unsigned word = 0x01010101u * byte;
    const size_t n16 = bytes / 16;
    const int ntail = (int)(bytes % 16);
    size_t blocks = (n16 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks == 0) blocks = 1;
    fill_kernel<<<dim3((unsigned)blocks), 256, 0, st>>>((uint4*)p, n16, (unsigned char*)p + n16 * 16, ntail, word);
}

}  // namespace fpdt
