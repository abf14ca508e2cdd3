// fp32 accuracy path, partial-result merge and fill kernels.
//
// The fp32 kernels compute the chunked attention on v_mfma_f32_16x16x4_f32 (fp32 operands, fp32
// accumulation) in the formulation of the bf16 kernels: forward and dQ hold S^T = K Q^T (a lane owns one
// query), dK/dV hold S = Q K^T (a lane owns one key), and the register-resident score tile is the next
// product's operand.  Their tensors are small (the accuracy configuration has 1K tokens), so what bounds
// them is the chain of one row tile and the number of launches: tiles have 16 rows (of 32 rows there are
// 64 at 1K tokens and two heads, a quarter of the compute units), the eight waves of a workgroup share a
// tile, each walking every eighth 32-row block of the other side, and their results meet in LDS; a call
// without FPDT_PAIRWISE is one forward and one backward launch.  At 1024 tokens, 2 heads, D = 64, chunks of 256, forward
// and backward: one wave per row with scalar dot products, pair by pair, 1799 us; 32-row tiles 110 us;
// this 64 us, with errors against fp64 below those of the scalar kernels in O, dQ, dK and dV (2.5e-7 .. 7.0e-7
// against 3.3e-7 .. 9.7e-7 over four shapes).
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
constexpr int BR = 32;   // rows of a block of the other side: two of the tiles' height

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

// acc^T [D x 16] += X^T [D x 16 rows] T [16 rows x 16 columns]: `t` is a score tile in accumulator layout
// (this lane: column lane % 16, rows 4 (lane / 16) + r), rows of X behind n_rows are not read.  `keep` has
// bit r set where t[r] counts; where it does not, t[r] is 0, but the row of X may hold infinities or NaN (a
// later key of this query), which 0 times it must not let through: those elements stay out of the product
// and are added one by one where they count.
template <int D>
__device__ __forceinline__ void add_rows(floatx4 (&acc)[D / 16], const floatx4& t, unsigned keep, const float* X, size_t pitch, int n_rows,
                                         int lane, float* park)
{
    const int g = lane >> 4, col = lane & 15;
    bool odd = false;
    if (n_rows <= 0) return;  // (wave-uniform)
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
        float x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = X[(size_t)(4 * g + r < n_rows ? 4 * g + r : 0) * pitch + 16 * db + col];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool fine = fabsf(x[r]) < INFINITY;
            odd |= !fine;
            acc[db] = mfma_f32(fine ? x[r] : 0.f, t[r], acc[db]);
        }
    }
    if (__builtin_expect(__any(odd), 0)) {
        // t by row through LDS; a NaN pattern that no arithmetic produces marks what does not count
#pragma unroll
        for (int r = 0; r < 4; ++r) park[(4 * g + r) * 16 + col] = (keep >> r) & 1 ? t[r] : __uint_as_float(0xffffdeadu);
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int row = 0; row < (n_rows < TR ? n_rows : TR); ++row) {
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

// Sum over the waves of a workgroup of acc^T [D x 16], and the result to out(d, column) for every element
// (17 floats per channel: the final reads, channel fastest, then fall into different banks)
template <int D, typename F>
__device__ __forceinline__ void sum_waves(const floatx4 (&acc)[D / 16], float* lds, F out)
{
    constexpr int ALL = D * 17;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    __syncthreads();
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) lds[w * ALL + (16 * db + 4 * g + r) * 17 + col] = acc[db][r];
    __syncthreads();
    // channel fastest over the threads: rows of the result are written in whole lines
    for (int e = threadIdx.x; e < D * TR; e += NW * 64) {
        const int d = e % D, c = e / D;
        float v = lds[d * 17 + c];
#pragma unroll
        for (int i = 1; i < NW; ++i) v += lds[i * ALL + d * 17 + c];
        out(d, c, v);
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
template <int D>
__global__ __launch_bounds__(64 * NW) void f32_fwd_kernel(F32FwdArgs a)
{
    constexpr int DB = D / 16, ALL = D * 17;
    __shared__ float lds[NW * ALL];
    __shared__ float ml[NW][2][TR];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    const int n_tiles = (int)((a.n_q + TR - 1) / TR);
    const int head = blockIdx.x % (unsigned)a.Hq, tile = n_tiles - 1 - (int)(blockIdx.x / (unsigned)a.Hq);  // longest first
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
    for (int64_t j0 = BR * w; j0 < need; j0 += BR * NW) {
        const int keys = (int)(a.n_k - j0 < BR ? a.n_k - j0 : BR);
        const float* k0 = a.K + j0 * k_pitch + (size_t)kvh * D;
        const float* v0 = a.V + j0 * k_pitch + (size_t)kvh * D;
        floatx4 s[2];
        unsigned keep[2] = {0, 0};
        float mx = -INFINITY;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            Rows<D> k;
            k.load(k0 + (size_t)(16 * b + col < keys ? 16 * b + col : keys - 1) * k_pitch, g);
            s[b] = dot_rows<D>(k, q);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = 16 * b + 4 * g + r;
                const bool on = key < keys && a.k_pos0 + j0 + key <= qpos;
                keep[b] |= (unsigned)on << r;
                s[b][r] = on ? a.scale * s[b][r] : -INFINITY;
                mx = fmaxf(mx, s[b][r]);
            }
        }
        const float m_new = fmaxf(m, max_over_rows(mx));
        // (every score of this wave so far may be -infinity, masked or overflowed: then 0 takes the maximum's
        // place, whatever was added is 0, and so stays what the next finite score rescales)
        const float m_ref = m_new > -INFINITY ? m_new : 0.f;
        const float alpha = expf(m - m_ref);
        l *= alpha;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[b][r] = (keep[b] >> r) & 1 ? expf(s[b][r] - m_ref) : 0.f;
                l += s[b][r];
            }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[db][r] *= alpha;
#pragma unroll
        for (int b = 0; b < 2; ++b) add_rows<D>(acc, s[b], keep[b], v0 + 16 * b * k_pitch, k_pitch, keys - 16 * b, lane, lds + w * ALL);
        m = m_new;
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
    sum_waves<D>(acc, lds, [&](int d, int c, float v) {
        if (c < rows) (final ? a.O : a.st_acc)[((size_t)(row0 + c) * a.Hq + head) * D + d] = v * ml[0][1][c];
    });
}

// One launch for both sides: the first workgroups own 16-query tiles (dQ), the others 16-key tiles (dK, dV:
// all query heads of the group).  Waves share the walk of a tile as in the forward.
template <int D>
__global__ __launch_bounds__(64 * NW) void f32_bwd_kernel(F32BwdArgs a, unsigned dq_blocks)
{
    constexpr int DB = D / 16, ALL = D * 17;
    __shared__ float lds[NW * ALL];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    const int group = a.Hq / a.Hkv;
    const size_t q_pitch = (size_t)a.Hq * D, k_pitch = (size_t)a.Hkv * D;
    float* park = lds + w * ALL;
    if (blockIdx.x < dq_blocks) {
        const int n_tiles = (int)((a.n_q + TR - 1) / TR);
        const int head = blockIdx.x % (unsigned)a.Hq, tile = n_tiles - 1 - (int)(blockIdx.x / (unsigned)a.Hq);
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
        for (int64_t j0 = BR * w; j0 < need; j0 += BR * NW) {
            const int keys = (int)(a.n_k - j0 < BR ? a.n_k - j0 : BR);
            const size_t k0 = j0 * k_pitch + (size_t)kvh * D;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const size_t kr = k0 + (size_t)(16 * b + col < keys ? 16 * b + col : keys - 1) * k_pitch;
                Rows<D> k;
                k.load(a.K + kr, g);
                floatx4 s = dot_rows<D>(k, q);
                k.load(a.V + kr, g);
                const floatx4 dp = dot_rows<D>(k, go);
                unsigned keep = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = 16 * b + 4 * g + r;
                    const bool on = key < keys && a.k_pos0 + j0 + key <= qpos;
                    keep |= (unsigned)on << r;
                    s[r] = on ? expf(a.scale * s[r] - lse) * (dp[r] - delta) : 0.f;
                }
                add_rows<D>(acc, s, keep, a.K + k0 + 16 * b * k_pitch, k_pitch, keys - 16 * b, lane, park);
            }
        }
        sum_waves<D>(acc, lds, [&](int d, int c, float v) {
            if (c < rows) {
                float* o = a.dQ + (row0 + c) * q_pitch + (size_t)head * D + d;
                *o = (a.accumulate ? *o : 0.f) + a.scale * v;
            }
        });
        return;
    }
    const unsigned blk = blockIdx.x - dq_blocks;
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
    for (int64_t t = w; t < blocks * group; t += NW) {
        const int head = kvh * group + (int)(t / blocks);
        const int64_t i0 = i_first + t % blocks * BR;
        const int rows = (int)(a.n_q - i0 < BR ? a.n_q - i0 : BR);
        const size_t q0 = i0 * q_pitch + (size_t)head * D;
        const float* lse = a.LSE + (size_t)head * a.row_stat_stride + i0;
        const float* delta = a.Delta + (size_t)head * a.row_stat_stride + i0;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const size_t qr = q0 + (size_t)(16 * b + col < rows ? 16 * b + col : rows - 1) * q_pitch;
            Rows<D> x;
            x.load(a.Q + qr, g);
            floatx4 s = dot_rows<D>(x, k);
            x.load(a.dO + qr, g);
            floatx4 ds = dot_rows<D>(x, v);
            unsigned keep = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = 16 * b + 4 * g + r;
                const bool on = row < rows && kpos <= a.q_pos0 + i0 + row;
                keep |= (unsigned)on << r;
                s[r] = on ? expf(a.scale * s[r] - lse[row < rows ? row : 0]) : 0.f;
                ds[r] = on ? s[r] * (ds[r] - delta[row < rows ? row : 0]) : 0.f;
            }
            add_rows<D>(dv, s, keep, a.dO + q0 + 16 * b * q_pitch, q_pitch, rows - 16 * b, lane, park);
            add_rows<D>(dk, ds, keep, a.Q + q0 + 16 * b * q_pitch, q_pitch, rows - 16 * b, lane, park);
        }
    }
    auto put = [&](float* out, float mul) {
        return [=](int d, int c, float x) {
            if (c < keys) {
                float* o = out + (key0 + c) * k_pitch + (size_t)kvh * D + d;
                *o = (a.accumulate ? *o : 0.f) + mul * x;
            }
        };
    };
    sum_waves<D>(dk, lds, put(a.dK, a.scale));
    sum_waves<D>(dv, lds, put(a.dV, 1.f));
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
    const dim3 grid(dq + (unsigned)((a.n_k + TR - 1) / TR * a.Hkv));
    if (a.D == 128) f32_bwd_kernel<128><<<grid, 64 * NW, 0, st>>>(a, dq);
    else if (a.D == 80) f32_bwd_kernel<80><<<grid, 64 * NW, 0, st>>>(a, dq);
    else f32_bwd_kernel<64><<<grid, 64 * NW, 0, st>>>(a, dq);
}

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
