// fp32 accuracy path, partial-result merge and fill kernels.
//
// The fp32 kernels compute the chunked attention on v_mfma_f32_32x32x2_f32 (fp32 operands, fp32
// accumulation) in the formulation of the bf16 kernels: forward and dQ hold S^T = K Q^T (a lane owns one
// query), dK/dV hold S = Q K^T (a lane owns one key), and the register-resident score tile is the next
// product's operand.  Their tensors are small (the accuracy configuration has 1K tokens), so what bounds
// them is the length of the chain of one 32-row tile and the number of launches: the waves of a
// workgroup share a tile, each walking every NW-th block of the other side, and their results meet in
// LDS; a dense call is one forward and one backward launch.  At 1024 tokens, 2 heads, D = 64, chunks
// of 256, one wave per row with scalar dot products, chunk pair by chunk pair, took 1799 us for forward
// and backward; this takes 110 us.
#include "fpdt_internal.h"
#include "mfma_tiles.h"

namespace fpdt {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// acc[32x32] += A[32x2] B[2x32]: lane l holds A[l % 32][l / 32] and B[l / 32][l % 32]
__device__ __forceinline__ floatx16 mfma_f32(float a, float b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Row operand of a product contracted over the channels: lane (row = lane % 32, h = lane / 32) holds
// channels 8 j + 4 h + 0..3, j = 0 .. D/8 - 1, of its row.  (Any order of the channels does, as both
// operands use the same.)
template <int D>
struct Rows {
    f32x4 v[D / 8];
    __device__ __forceinline__ void load(const float* row, int half)
    {
#pragma unroll
        for (int j = 0; j < D / 8; ++j) v[j] = *reinterpret_cast<const f32x4*>(row + 8 * j + 4 * half);
    }
};
template <int D>
__device__ __forceinline__ floatx16 dot_rows(const Rows<D>& a, const Rows<D>& b)
{
    floatx16 s = {};
#pragma unroll
    for (int j = 0; j < D / 8; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) s = mfma_f32(a.v[j][c], b.v[j][c], s);
    __builtin_amdgcn_sched_barrier(0);  // the next product's loads do not fit beside this one's operands
    return s;
}

// acc^T [D x 32] += X^T [D x 32 rows] T [32 rows x 32 columns]: `t` is a score tile in accumulator layout
// (this lane: column lane % 32, rows 8 (r / 4) + 4 (lane / 32) + r % 4), rows of X behind n_rows are not
// read.  `keep` has bit r set where t[r] counts; where it does not, t[r] is 0, but the row of X may hold
// infinities or NaN (a later key of this query), which 0 times it must not let through: those elements
// stay out of the product and are added one by one where they count.
template <int D>
__device__ __forceinline__ void add_rows(floatx16 (&acc)[(D + 31) / 32], const floatx16& t, unsigned keep, const float* X, size_t pitch,
                                         int n_rows, int lane, float* park)
{
    constexpr int DB = (D + 31) / 32;
    const int half = lane >> 5, col = lane & 31;
    bool odd = false;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        const int d = 32 * db + col < D ? 32 * db + col : D - 1;  // (channels behind D are not stored)
        float x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 8 * (r >> 2) + 4 * half + (r & 3);
            x[r] = X[(size_t)(row < n_rows ? row : 0) * pitch + d];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const bool fine = fabsf(x[r]) < INFINITY;
            odd |= !fine;
            acc[db] = mfma_f32(fine ? x[r] : 0.f, t[r], acc[db]);
        }
    }
    if (__builtin_expect(__any(odd), 0)) {
        // t by row through LDS; a NaN pattern that no arithmetic produces marks what does not count
#pragma unroll
        for (int r = 0; r < 16; ++r) park[(8 * (r >> 2) + 4 * half + (r & 3)) * 32 + col] = (keep >> r) & 1 ? t[r] : __uint_as_float(0xffffdeadu);
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int row = 0; row < n_rows; ++row) {
            const float p = park[row * 32 + col];
            const bool on = __float_as_uint(p) != 0xffffdeadu;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int d = 32 * db + 8 * q + 4 * half;
                    const f32x4 v = *reinterpret_cast<const f32x4*>(X + (size_t)row * pitch + (d < D ? d : 0));
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (on && !(fabsf(v[e]) < INFINITY)) acc[db][4 * q + e] += p * v[e];
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Sum over the waves of a workgroup of acc^T [D x 32], and the result to out(d, column) for every element
// (33 floats per channel: the final reads, channel fastest, then fall into different banks)
template <int D, int NW, typename F>
__device__ __forceinline__ void sum_waves(const floatx16 (&acc)[(D + 31) / 32], float* lds, F out)
{
    constexpr int DB = (D + 31) / 32, ALL = DB * 32 * 33;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5, col = lane & 31;
    __syncthreads();
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) lds[w * ALL + (32 * db + 8 * (r >> 2) + 4 * half + (r & 3)) * 33 + col] = acc[db][r];
    __syncthreads();
    // channel fastest over the threads: rows of the result are written in whole lines
    for (int e = threadIdx.x; e < D * 32; e += NW * 64) {
        const int d = e % D, c = e / D;
        float v = lds[d * 33 + c];
#pragma unroll
        for (int i = 1; i < NW; ++i) v += lds[i * ALL + d * 33 + c];
        out(d, c, v);
    }
}

template <int D> constexpr int f32_waves() { return D > 64 ? 4 : 8; }  // D > 64: one wave per SIMD, for its registers

// Workgroup = one 32-query tile of one head; wave w folds key blocks w, w + NW, .. into its own (max, sum,
// un-normalised output), wave 0 starting from the carried state; they are merged at the end.
template <int D>
__global__ __launch_bounds__(64 * f32_waves<D>()) void f32_fwd_kernel(F32FwdArgs a)
{
    constexpr int NW = f32_waves<D>(), DB = (D + 31) / 32, ALL = DB * 32 * 33;
    __shared__ float lds[NW * ALL];
    __shared__ float ml[NW][2][32];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5, col = lane & 31;
    const int n_tiles = (int)((a.n_q + 31) / 32);
    const int head = blockIdx.x % (unsigned)a.Hq, tile = n_tiles - 1 - (int)(blockIdx.x / (unsigned)a.Hq);  // longest first
    const int kvh = head / (a.Hq / a.Hkv);
    const int64_t row0 = (int64_t)tile * 32;
    const int rows = (int)(a.n_q - row0 < 32 ? a.n_q - row0 : 32);
    const size_t q_pitch = (size_t)a.Hq * D, k_pitch = (size_t)a.Hkv * D;
    const float* q0 = a.Q + row0 * q_pitch + (size_t)head * D;
    const int64_t qpos = a.q_pos0 + row0 + (col < rows ? col : rows - 1);
    Rows<D> q;
    q.load(q0 + (size_t)(col < rows ? col : rows - 1) * q_pitch, half);

    float m = -INFINITY, l = 0.f;
    floatx16 acc[DB] = {};
    if (w == 0 && !(a.flags & SWEEP_INIT) && col < rows) {
        const size_t at = (size_t)(row0 + col) * a.Hq + head;
        m = a.st_ml[2 * at];
        l = half == 0 ? a.st_ml[2 * at + 1] : 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int d = 32 * db + 8 * (r >> 2) + 4 * half + (r & 3);
                if (d < D) acc[db][r] = a.st_acc[at * D + d];
            }
    }
    int64_t need = a.q_pos0 + row0 + rows - a.k_pos0;  // keys at positions <= the last query's
    if (need > a.n_k) need = a.n_k;
    for (int64_t j0 = 32 * w; j0 < need; j0 += 32 * NW) {
        const int keys = (int)(a.n_k - j0 < 32 ? a.n_k - j0 : 32);
        const float* k0 = a.K + j0 * k_pitch + (size_t)kvh * D;
        Rows<D> k;
        k.load(k0 + (size_t)(col < keys ? col : keys - 1) * k_pitch, half);
        floatx16 s = dot_rows<D>(k, q);
        unsigned keep = 0;
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = 8 * (r >> 2) + 4 * half + (r & 3);
            const bool on = key < keys && a.k_pos0 + j0 + key <= qpos;
            keep |= (unsigned)on << r;
            s[r] = on ? a.scale * s[r] : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        mx = fmaxf(mx, xor32(mx));
        const float m_new = fmaxf(m, mx);
        const float alpha = m_new > -INFINITY ? expf(m - m_new) : 1.f;  // (no key of this row yet: nothing to rescale)
        l *= alpha;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s[r] = (keep >> r) & 1 ? expf(s[r] - m_new) : 0.f;
            l += s[r];
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] *= alpha;
        add_rows<D>(acc, s, keep, a.V + j0 * k_pitch + (size_t)kvh * D, k_pitch, keys, lane, lds + w * ALL);
        m = m_new;
    }
    l += xor32(l);
    if (half == 0) {
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
        for (int r = 0; r < 16; ++r) acc[db][r] = empty ? 0.f : acc[db][r] * mine;
    const bool final = a.flags & SWEEP_FINAL;
    __syncthreads();
    if (w == 0 && half == 0) {
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
    sum_waves<D, NW>(acc, lds, [&](int d, int c, float v) {
        if (c < rows) (final ? a.O : a.st_acc)[((size_t)(row0 + c) * a.Hq + head) * D + d] = v * ml[0][1][c];
    });
}

// One launch for both sides: the first workgroups own 32-query tiles (dQ), the others 32-key tiles (dK, dV:
// all query heads of the group).  Waves share the walk of a tile as in the forward.
template <int D>
__global__ __launch_bounds__(64 * f32_waves<D>()) void f32_bwd_kernel(F32BwdArgs a, unsigned dq_blocks)
{
    constexpr int NW = f32_waves<D>(), DB = (D + 31) / 32, ALL = DB * 32 * 33;
    __shared__ float lds[NW * ALL];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5, col = lane & 31;
    const int g = a.Hq / a.Hkv;
    const size_t q_pitch = (size_t)a.Hq * D, k_pitch = (size_t)a.Hkv * D;
    float* park = lds + w * ALL;
    if (blockIdx.x < dq_blocks) {
        const int n_tiles = (int)((a.n_q + 31) / 32);
        const int head = blockIdx.x % (unsigned)a.Hq, tile = n_tiles - 1 - (int)(blockIdx.x / (unsigned)a.Hq);
        const int kvh = head / g;
        const int64_t row0 = (int64_t)tile * 32;
        const int rows = (int)(a.n_q - row0 < 32 ? a.n_q - row0 : 32), mine = col < rows ? col : rows - 1;
        const int64_t qpos = a.q_pos0 + row0 + mine;
        Rows<D> q, go;
        q.load(a.Q + (row0 + mine) * q_pitch + (size_t)head * D, half);
        go.load(a.dO + (row0 + mine) * q_pitch + (size_t)head * D, half);
        const float lse = a.LSE[(size_t)head * a.row_stat_stride + row0 + mine];
        const float delta = a.Delta[(size_t)head * a.row_stat_stride + row0 + mine];
        floatx16 acc[DB] = {};
        int64_t need = a.q_pos0 + row0 + rows - a.k_pos0;
        if (need > a.n_k) need = a.n_k;
        for (int64_t j0 = 32 * w; j0 < need; j0 += 32 * NW) {
            const int keys = (int)(a.n_k - j0 < 32 ? a.n_k - j0 : 32);
            const size_t k0 = j0 * k_pitch + (size_t)kvh * D, kr = k0 + (size_t)(col < keys ? col : keys - 1) * k_pitch;
            Rows<D> k;
            k.load(a.K + kr, half);
            floatx16 s = dot_rows<D>(k, q);
            k.load(a.V + kr, half);
            const floatx16 dp = dot_rows<D>(k, go);
            unsigned keep = 0;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = 8 * (r >> 2) + 4 * half + (r & 3);
                const bool on = key < keys && a.k_pos0 + j0 + key <= qpos;
                keep |= (unsigned)on << r;
                s[r] = on ? expf(a.scale * s[r] - lse) * (dp[r] - delta) : 0.f;
            }
            add_rows<D>(acc, s, keep, a.K + k0, k_pitch, keys, lane, park);
        }
        sum_waves<D, NW>(acc, lds, [&](int d, int c, float v) {
            if (c < rows) {
                float* o = a.dQ + (row0 + c) * q_pitch + (size_t)head * D + d;
                *o = (a.accumulate ? *o : 0.f) + a.scale * v;
            }
        });
        return;
    }
    const unsigned b = blockIdx.x - dq_blocks;
    const int kvh = b % (unsigned)a.Hkv;
    const int64_t key0 = (int64_t)(b / (unsigned)a.Hkv) * 32;  // first keys first: theirs is the longest walk
    const int keys = (int)(a.n_k - key0 < 32 ? a.n_k - key0 : 32), mine = col < keys ? col : keys - 1;
    const int64_t kpos = a.k_pos0 + key0 + mine;
    Rows<D> k, v;
    k.load(a.K + (key0 + mine) * k_pitch + (size_t)kvh * D, half);
    v.load(a.V + (key0 + mine) * k_pitch + (size_t)kvh * D, half);
    floatx16 dk[DB] = {}, dv[DB] = {};
    int64_t i_first = a.k_pos0 + key0 - a.q_pos0;  // first query row that attends the tile's first key
    if (i_first < 0) i_first = 0;
    const int64_t blocks = i_first < a.n_q ? (a.n_q - i_first + 31) / 32 : 0;
    for (int64_t t = w; t < blocks * g; t += NW) {
        const int head = kvh * g + (int)(t / blocks);
        const int64_t i0 = i_first + t % blocks * 32;
        const int rows = (int)(a.n_q - i0 < 32 ? a.n_q - i0 : 32);
        const size_t q0 = i0 * q_pitch + (size_t)head * D, qr = q0 + (size_t)(col < rows ? col : rows - 1) * q_pitch;
        const float* lse = a.LSE + (size_t)head * a.row_stat_stride + i0;
        const float* delta = a.Delta + (size_t)head * a.row_stat_stride + i0;
        Rows<D> x;
        x.load(a.Q + qr, half);
        floatx16 s = dot_rows<D>(x, k);
        x.load(a.dO + qr, half);
        floatx16 ds = dot_rows<D>(x, v);
        unsigned keep = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = 8 * (r >> 2) + 4 * half + (r & 3);
            const bool on = row < rows && kpos <= a.q_pos0 + i0 + row;
            keep |= (unsigned)on << r;
            s[r] = on ? expf(a.scale * s[r] - lse[row < rows ? row : 0]) : 0.f;
            ds[r] = on ? s[r] * (ds[r] - delta[row < rows ? row : 0]) : 0.f;
        }
        add_rows<D>(dv, s, keep, a.dO + q0, q_pitch, rows, lane, park);
        add_rows<D>(dk, ds, keep, a.Q + q0, q_pitch, rows, lane, park);
    }
    auto put = [&](float* out, float mul) {
        return [=](int d, int c, float x) {
            if (c < keys) {
                float* o = out + (key0 + c) * k_pitch + (size_t)kvh * D + d;
                *o = (a.accumulate ? *o : 0.f) + mul * x;
            }
        };
    };
    sum_waves<D, NW>(dk, lds, put(a.dK, a.scale));
    sum_waves<D, NW>(dv, lds, put(a.dV, 1.f));
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
    const dim3 grid((unsigned)((a.n_q + 31) / 32 * a.Hq));
    if (a.D == 128) f32_fwd_kernel<128><<<grid, 64 * f32_waves<128>(), 0, st>>>(a);
    else if (a.D == 80) f32_fwd_kernel<80><<<grid, 64 * f32_waves<80>(), 0, st>>>(a);
    else f32_fwd_kernel<64><<<grid, 64 * f32_waves<64>(), 0, st>>>(a);
}

void launch_f32_bwd(const F32BwdArgs& a, hipStream_t st)
{
    const unsigned dq = (unsigned)((a.n_q + 31) / 32 * a.Hq);
    const dim3 grid(dq + (unsigned)((a.n_k + 31) / 32 * a.Hkv));
    if (a.D == 128) f32_bwd_kernel<128><<<grid, 64 * f32_waves<128>(), 0, st>>>(a, dq);
    else if (a.D == 80) f32_bwd_kernel<80><<<grid, 64 * f32_waves<80>(), 0, st>>>(a, dq);
    else f32_bwd_kernel<64><<<grid, 64 * f32_waves<64>(), 0, st>>>(a, dq);
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
