// Forward chunk sweep on bf16 MFMA (Sec. 4.1: query chunk against key/value chunks with
// online-softmax accumulation; causal mask only where the key range reaches the queries).
//
// Formulation: the score tile is computed transposed, S^T = K Q^T (keys are MFMA rows,
// queries are MFMA columns).  In the 32x32 accumulator layout a lane then owns ONE query
// (column lane%32) and 16 keys per 32-key block, so the running max of a query needs a single
// exchange between lanes l and l+32, the running sum none until the epilogue, and the
// exponentiated tile -- still in registers -- is directly the B operand of O^T += V^T P^T.
// K arrives as NAT fragments, V as TR fragments (fpdt_internal.h), or both from their tensors (RAW below); Q is loaded
// once and stays in registers.
//
// Workgroup = 8 waves (two per SIMD, so one wave's softmax arithmetic runs under the other's
// MFMAs; 4 where a launch of one key group would otherwise leave half of the chip idle, sweep_waves), each wave owns 32 query
// rows of one head and at most 256 registers.  The K/V tiles travel
// global -> LDS directly (no register staging) through a ring filled ahead.  KG = 1: the waves own 256
// query rows and share 64-key tiles.  KG = 2, 4: 128 or 64 query rows, the waves of one row block take
// every KG-th 32-key block and merge their (max, sum, output) through LDS at the end, for launches whose
// row tiles are too few to fill the chip or whose longest row tile decides (sweep_key_groups).
#include "fpdt_internal.h"
#include "mfma_tiles.h"

namespace fpdt {

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

struct FwdKernelArgs {
    const uint16_t* Q;
    const u32x4* Knat;
    const u32x4* Vtr;
    const uint16_t* K;  // RAW: the tensors themselves, [n_keys, Hkv, D]
    const uint16_t* V;
    int64_t kv_pitch;   // elements between their rows
    int ahead_rows;     // of K and V that each of the first workgroups of a head reads ahead (0: none)
    int64_t kv_head_stride_blocks;
    uint16_t* O;
    float* LSE;
    int64_t lse_stride;
    float* st_acc;
    float* st_ml;
    int64_t q_pos0, k_pos0;
    int n_q, n_keys;
    int Hq, g, flags;
    float c;  // scale * log2(e)
};

// RAW: K and V come from their row-major tensors instead of packed fragments.  A 32-key block is copied row by row, 16-byte
// piece q of row r at position q ^ swz(r) of its row, swz(r) = 4 (r % 4) + (r / 4) % 4 (D = 64: 4 (r / 2 % 2) + (r / 4) %
// 4; D = 80: rows of ten pieces as they are): the lanes that a fragment read serves at a time, and the four rows of a
// transposing read, lie in different banks.  V's operand is then read with transposing loads, two for one plain
// read.  For short sequences, where the packing launch costs more than these reads (sweep_reads_tensors, launch_rules.h).
template <int D, int KG, int NWAVE, bool RAW>
__global__ __launch_bounds__(NWAVE * 64, 2) void fwd_sweep_kernel(FwdKernelArgs p)
{
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int KB = KG == 1 ? 2 : 1;     // 32-key blocks of a wave per tile
    constexpr int NB = KG * KB, BK = NB * 32;  // blocks and keys per LDS tile
    constexpr int NQ = NWAVE / KG, BQ = NQ * 32;  // row blocks and query rows per workgroup
    constexpr int RING = KG == 4 || NWAVE < 8 ? 2 : 3;  // (a tile of 128 keys: 64 KiB at D = 128; four waves: room for two workgroups)
    constexpr int PF = RING - 1;            // tiles in flight ahead of the one being computed
    constexpr int K_U4 = NB * DT * 64;      // u32x4 per K tile
    constexpr int VF = RAW ? DT : 2 * DB;   // 1 KiB copies of V per 32-key block
    constexpr int V_U4 = NB * VF * 64;      // u32x4 per V tile
    constexpr int T_U4 = K_U4 + V_U4;
    constexpr int KFRAG = NB * DT, NFRAG = KFRAG + NB * VF;  // 1 KiB copies per tile
    constexpr int PAD = RAW && DP > D ? 4 : 0;  // the last row's padded channels are read from behind it
    // KG = 1: one LDS array per ring slot; otherwise one for all, which the final merge uses again
    __shared__ u32x4 ring_a[KG == 1 ? T_U4 : RING * T_U4 + PAD], ring_b[KG == 1 ? T_U4 : 1], ring_c[KG == 1 ? T_U4 : 1];
    u32x4* const ring0 = ring_a;
    u32x4* const ring1 = KG == 1 ? ring_b : ring_a + T_U4;
    u32x4* const ring2 = KG == 1 ? ring_c : ring_a + (RING - 1) * T_U4;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int half = lane >> 5, col = lane & 31;
    const int qb = KG == 1 ? w : wu % NQ, kg = KG == 1 ? 0 : wu / NQ;  // this wave's row block and its share of the key blocks
    const int head = blockIdx.x % p.Hq;
    const int n_qt = p.n_q / BQ;
    const int qt = n_qt - 1 - (int)(blockIdx.x / p.Hq);  // heaviest (latest) tiles first
    const int kvh = head / p.g;
    const int q0 = qt * BQ;       // first row of the workgroup within the launch
    const int qw0 = q0 + qb * 32;  // first row of this wave

    // keys this workgroup needs: positions <= last query position
    const int64_t last_q_pos = p.q_pos0 + q0 + BQ - 1;
    int64_t need = last_q_pos - p.k_pos0 + 1;
    if (need > p.n_keys) need = p.n_keys;
    const int n_tiles = (int)((need + BK - 1) / BK);

    const u32x4* kbase = p.Knat + (size_t)kvh * p.kv_head_stride_blocks * (DT * 64);
    const u32x4* vbase = p.Vtr + (size_t)kvh * p.kv_head_stride_blocks * (2 * DB * 64);

    // RAW: this lane's byte offset within copy c of a 32-key block, and its reads within a block
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef short short8v __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
    typedef __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
    constexpr int PPR = D / 8, ROW = 2 * D;  // pieces and bytes of a row
    const unsigned pitch = RAW ? (unsigned)p.kv_pitch * 2u : 0u;
    auto swz = [](int r) { return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : D == 64 ? (((r >> 1) & 1) << 2) | ((r >> 2) & 3) : 0; };
    auto raw_offset = [&](int c) {
        const int piece = 64 * c + lane, r = D == 80 ? (piece * 6554) >> 16 : piece / PPR;
        return (unsigned)r * pitch + 16u * (unsigned)((piece - r * PPR) ^ swz(r));
    };
    const unsigned raw_off = RAW && D != 80 ? raw_offset(wu % DT) : 0u;  // (every copy of a wave is the same one of its block)
    const unsigned k_rd = (unsigned)(col * ROW + 16 * (half ^ swz(col)));
    unsigned v_rd[2];
    {
        const int grp = lane >> 4, h = grp >> 1, dblk = grp & 1, e = (lane & 15) >> 2, x = lane & 3;
#pragma unroll
        for (int I = 0; I < 2; ++I) {
            const int r = 8 * I + 4 * h + e;
            v_rd[I] = (unsigned)(r * ROW + 16 * ((2 * dblk + (x >> 1)) ^ swz(r)) + 8 * (x & 1));
        }
    }

    // Copy tile `it` into ring slot `slot`: wave w moves fragments w, w+8, ...
    auto issue = [&](int it, u32x4* slot) {
        if constexpr (RAW) {
            static_assert(D == 80 || (KFRAG % NWAVE == 0 && NWAVE % DT == 0), "a wave's copies are the same one of every block");
            const unsigned lds = lds_address(slot);
            const uint64_t row0 = (uint64_t)it * BK * pitch + (uint64_t)kvh * ROW;
#pragma unroll
            for (int f0 = 0; f0 < NFRAG; f0 += NWAVE) {
                const int f = f0 + wu;
                if (f0 + NWAVE <= NFRAG || f < NFRAG) {
                    const bool of_k = f < KFRAG;
                    const int fb = of_k ? f : f - KFRAG, blk = fb / DT, c = fb - blk * DT;
                    const uint64_t src = (uint64_t)(uintptr_t)(of_k ? p.K : p.V) + row0 + (uint64_t)(32 * blk) * pitch;
                    frag_to_lds_at(uniform(src), lds + 1024u * (unsigned)f, (int)(D == 80 ? raw_offset(c) : raw_off));
                }
            }
            return;
        }
        const u32x4* ksrc = kbase + (size_t)it * K_U4;
        const u32x4* vsrc = vbase + (size_t)it * V_U4;
#pragma unroll
        for (int f0 = 0; f0 < NFRAG; f0 += NWAVE) {
            const int f = f0 + wu;
            if (f0 + NWAVE <= NFRAG || f < NFRAG) {
                const u32x4* src = f < KFRAG ? ksrc + f * 64 : vsrc + (f - KFRAG) * 64;
                frag_to_lds(src, slot + f * 64, lane);
            }
        }
    };

    // Q fragments (B operand of S^T = K Q^T): lane (col, half) holds Q[row][16t + 8 half + e]
    bf16x8 qf[DT];
    {
        const uint16_t* qrow = p.Q + ((size_t)(qw0 + col) * p.Hq + head) * D + 8 * half;
#pragma unroll
        for (int t = 0; t < DT; ++t) qf[t] = as_bf16x8(*reinterpret_cast<const u32x4*>(qrow + 16 * t));
    }

    floatx16 acc[DB];
    float m_run, l_run;  // l_run is this lane's partial sum (its 16 keys per block)
    const size_t slot = ((size_t)(qw0 / 32) * p.Hq + head) * KG + kg;  // every key group carries its own state
    float* sa = p.st_acc + slot * (size_t)(DB * 16 * 64);
    float* sm = p.st_ml + slot * (size_t)(2 * 64);
    if (p.flags & SWEEP_INIT) {
        m_run = -INFINITY;
        l_run = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    } else {
        m_run = sm[lane];
        l_run = sm[64 + lane];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = sa[(db * 16 + r) * 64 + lane];
    }

    if (n_tiles > 0) issue(0, ring0);
    if (PF > 1 && n_tiles > 1) issue(1, ring1);
    if constexpr (RAW && KG == 4) {
        // The packing launch also brought K and V into the caches, all of them at once.  With one tile in flight a workgroup
        // would fetch them tile after tile, each at the latency of HBM (inputs that no cache holds: 8 / 2 heads, D = 128, 2K
        // 31.4 us, 8 / 8, D = 64, 4K 46.0; packed 28.5, 35.0; this 27.1, 32.6).  So the workgroups of a head that start
        // first read a word of every line of its K and V between them, in the shadow of the first tile.
        constexpr int LINES = D == 64 ? 1 : 2;  // of 128 bytes, of a row of the head: those of its first and its last word
        const int row0 = (n_qt - 1 - qt) * p.ahead_rows, words = (p.n_keys - row0 < p.ahead_rows ? p.n_keys - row0 : p.ahead_rows) * LINES;
        if (words > 0) {
            unsigned seen = 0;
#pragma unroll 1
            for (int i = tid; i < words; i += NWAVE * 64) {
                const size_t at = (size_t)(row0 + i / LINES) * p.kv_pitch + (size_t)kvh * D + (i % LINES ? D - 2 : 0);
                seen |= *reinterpret_cast<const unsigned*>(p.K + at) | *reinterpret_cast<const unsigned*>(p.V + at);
            }
            asm volatile("" ::"v"(seen));
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    const int64_t qpos_first = p.q_pos0 + qw0;  // first / last query position of this wave
    const int64_t qpos_last = qpos_first + 31;
    const int64_t qpos = qpos_first + col;
    const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

    // One tile: compute on slot `ks`, prefetch tile it+PF into slot `pf_slot`.
    auto tile = [&](int it, const u32x4* ks, u32x4* pf_slot) {
        if (it + PF < n_tiles) issue(it + PF, pf_slot);
        const u32x4* vs = ks + K_U4;
        const int kb0 = kg * KB;  // this wave's first block within the tile
        const int64_t key0 = p.k_pos0 + (int64_t)it * BK + 32 * kb0;  // position of its first key

        if (key0 <= qpos_last) {  // wave-uniform: tile not entirely above this wave's diagonal
            // ---- S^T = K Q^T for the whole tile: all K fragments are requested up front so
            // that the MFMA chain never waits on LDS latency ----
            bf16x8 kfr[KB][DT];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    if constexpr (RAW) {
                        const unsigned at = D == 80 ? k_rd + 32u * (unsigned)t : k_rd ^ (32u * (unsigned)t);
                        kfr[kb][t] = as_bf16x8(*(lds_u32x4_ptr)(uintptr_t)(lds_address(ks) + 1024u * (unsigned)((kb0 + kb) * DT) + at));
                    } else {
                        kfr[kb][t] = as_bf16x8(ks[((kb0 + kb) * DT + t) * 64 + lane]);
                    }
                }
            floatx16 s[KB];
#pragma unroll
            for (int t = 0; t < DT; ++t)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) s[kb] = mfma32(kfr[kb][t], qf[t], t == 0 ? zero : s[kb]);
            __builtin_amdgcn_sched_group_barrier(0x100, KB * DT, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, KB * DT, 0);
            // V fragments are requested now and arrive under the softmax arithmetic
            bf16x8 vfr[KB][2][DB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        if constexpr (RAW) {
                            const unsigned blk = lds_address(vs) + 1024u * (unsigned)((kb0 + kb) * DT) + (unsigned)(16 * s2 * ROW);
                            auto at = [&](int I) { return blk + (D == 80 ? v_rd[I] + 64u * (unsigned)db : v_rd[I] ^ (64u * (unsigned)db)); };
                            const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)at(0));
                            const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)at(1));
                            const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                            vfr[kb][s2][db] = __builtin_bit_cast(bf16x8, both);
                        } else {
                            vfr[kb][s2][db] = as_bf16x8(vs[(((kb0 + kb) * 2 + s2) * DB + db) * 64 + lane]);
                        }
                    }
            __builtin_amdgcn_sched_group_barrier(0x100, KB * 2 * DB * (RAW ? 2 : 1), 0);
            // ---- online softmax, one query per lane ----
            if (key0 + 32 * KB - 1 > qpos_first) {  // wave-uniform: the tile straddles the diagonal
                // key index within the tile vs this lane's query, in 32 bits: a key is masked
                // when 32 kb + 8 (r / 4) + r % 4 + 4 half > qpos - key0
                int64_t d = qpos - key0;
                d = d < -1 ? -1 : d > 32 * KB ? 32 * KB : d;
                const int rel = (int)d - 4 * half;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (32 * kb + 8 * (r >> 2) + (r & 3) > rel) s[kb][r] = -INFINITY;
            }
            // The running maximum is only a reference point: any value gives the same O and LSE as
            // long as nothing overflows.  So the tile is exponentiated against the reference it
            // found, optimistically, and no maximum is taken at all; the row sums that are needed
            // anyway tell when that was wrong: every probability is at most the partial sum it
            // went into, so a sum within REF_LIMIT (far inside the range of bf16 and of the fp32
            // sums) proves that no probability exceeded it.  A sum beyond it -- or infinite, or not
            // a number, as on a row's first tile, where the reference is still -inf -- sends the
            // whole wave through the exact path below (true maximum, rescale, exponentiate again):
            // a row's first tile, and later only when its maximum rises by more than 14 in log2.
            constexpr float REF_LIMIT = 16384.f;
            bf16x8 pf[KB][2];
            float lsum = 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                floatx16 e;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    e[r] = __builtin_amdgcn_exp2f(fmaf(s[kb][r], p.c, -m_run));
                    lsum += e[r];
                }
                pf[kb][0] = pack_half<0>(e);
                pf[kb][1] = pack_half<1>(e);
            }
            if (__any(!(lsum <= REF_LIMIT))) {
                float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int r = (kb == 0 ? 2 : 0); r < 16; r += 2) mx = fmaxf(fmaxf(mx, s[kb][r]), s[kb][r + 1]);
                mx = fmaxf(mx, xor32(mx));
                const float mc = mx * p.c;
                const float m_new = mc > m_run ? mc : m_run;  // (a lane whose keys are all masked keeps its reference)
                // (KG > 1: a row may have had no key in this wave's blocks yet; its reference stays at -inf,
                // and 0 takes its place in the exponents)
                const float m_exp = KG > 1 && m_new == -INFINITY ? 0.f : m_new;
                const float alpha = __builtin_amdgcn_exp2f(m_run - m_exp);  // 0 on a row's first tile, 1 where nothing moved
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[db][r] *= alpha;
                m_run = m_new;
                lsum = 0.f;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    floatx16 e;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        e[r] = __builtin_amdgcn_exp2f(fmaf(s[kb][r], p.c, -m_exp));
                        lsum += e[r];
                    }
                    pf[kb][0] = pack_half<0>(e);
                    pf[kb][1] = pack_half<1>(e);
                }
            }
            l_run += lsum;
            // ---- O^T += V^T P^T ----
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int db = 0; db < DB; ++db)
                        acc[db] = mfma32(vfr[kb][s2][db], pf[kb][s2], acc[db]);
        }
        // tile it+1 must have landed; the loads of tile it+PF issued above may stay in flight
        if (it + PF < n_tiles) wait_vmem_at_most<(PF - 1) * (NFRAG / NWAVE)>();
        else wait_vmem_at_most<0>();
        barrier_no_fence();
    };
    if (RING == 3) {
        for (int it = 0; it < n_tiles; it += 3) {
            tile(it, ring0, ring2);
            if (it + 1 < n_tiles) tile(it + 1, ring1, ring0);
            if (it + 2 < n_tiles) tile(it + 2, ring2, ring1);
        }
    } else {
        for (int it = 0; it < n_tiles; it += 2) {
            tile(it, ring0, ring1);
            if (it + 1 < n_tiles) tile(it + 1, ring1, ring0);
        }
    }

    if (KG > 1 && (p.flags & SWEEP_FINAL)) {
        // Merge into the waves of kg = 0.  (Every copy has landed and every wave is past the last barrier:
        // nobody reads the ring any more.)
        constexpr int PART = (DB * 16 + 2) * 64;  // floats of a wave
        static_assert(KG == 1 || (NWAVE - NQ) * PART * 4 <= RING * T_U4 * 16, "the ring holds the parts");
        float* part = reinterpret_cast<float*>(ring_a);
        if (kg > 0) {
            float* mine = part + (size_t)((kg - 1) * NQ + qb) * PART + lane;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[(db * 16 + r) * 64] = acc[db][r];
            mine[DB * 16 * 64] = m_run;
            mine[(DB * 16 + 1) * 64] = l_run;
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int i = 1; i < KG; ++i) {
            const float* other = part + (size_t)((i - 1) * NQ + qb) * PART + lane;
            const float m_o = other[DB * 16 * 64], l_o = other[(DB * 16 + 1) * 64];
            const float m_new = m_o > m_run ? m_o : m_run;  // finite: this wave saw the first key of every row
            const float mine = __builtin_amdgcn_exp2f(m_run - m_new), theirs = __builtin_amdgcn_exp2f(m_o - m_new);
            l_run = l_run * mine + l_o * theirs;
            m_run = m_new;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] = acc[db][r] * mine + other[(db * 16 + r) * 64] * theirs;
        }
    }

    // ---- epilogue ----
    if (p.flags & SWEEP_FINAL) {
        const float l_tot = l_run + xor32(l_run);
        const float inv = 1.f / l_tot;
        const int row = qw0 + col;
        uint16_t* orow = p.O + ((size_t)row * p.Hq + head) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
                const int d = 32 * db + 8 * a4 + 4 * half;
                if (d < D) {
                    floatx4 v;
#pragma unroll
                    for (int b = 0; b < 4; ++b) v[b] = acc[db][4 * a4 + b] * inv;
                    *reinterpret_cast<bf16x4*>(orow + d) = __builtin_convertvector(v, bf16x4);
                }
            }
        if (half == 0) p.LSE[(size_t)head * p.lse_stride + row] = (m_run + __builtin_log2f(l_tot)) * LN2;
    } else {
        sm[lane] = m_run;
        sm[64 + lane] = l_run;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) sa[(db * 16 + r) * 64 + lane] = acc[db][r];
    }
}

}  // namespace

size_t fwd_state_acc_bytes(int64_t n_q, int Hq, int D, int key_groups)
{
    return (size_t)n_q * Hq * dpad(D) * sizeof(float) * key_groups;
}
size_t fwd_state_ml_bytes(int64_t n_q, int Hq, int D, int key_groups)
{
    (void)D;
    return (size_t)n_q * Hq * 2 * 2 * sizeof(float) * key_groups;  // (m, l) for both half-lanes of a row
}

void launch_fwd_sweep(const FwdArgs& a, hipStream_t st)
{
    FwdKernelArgs k;
    k.Q = static_cast<const uint16_t*>(a.Q);
    k.Knat = static_cast<const u32x4*>(a.Knat);
    k.Vtr = static_cast<const u32x4*>(a.Vtr);
    k.K = static_cast<const uint16_t*>(a.K);
    k.V = static_cast<const uint16_t*>(a.V);
    k.kv_pitch = (int64_t)a.Hkv * a.D;
    k.kv_head_stride_blocks = a.kv_head_stride_blocks;
    k.O = static_cast<uint16_t*>(a.O);
    k.LSE = a.LSE;
    k.lse_stride = a.lse_stride;
    k.st_acc = a.st_acc;
    k.st_ml = a.st_ml;
    k.q_pos0 = a.q_pos0;
    k.k_pos0 = a.k_pos0;
    k.n_q = (int)a.n_q;
    k.n_keys = (int)a.n_keys;
    k.Hq = a.Hq;
    k.g = a.Hq / a.Hkv;
    k.flags = a.flags;
    k.c = a.scale * LOG2E;
    // 256 workgroups start at once.  (Up to 768 keys there are too few tiles for it; two key groups have two tiles in flight and 16
    // heads and more: reading ahead gained nothing there and cost up to 8%.)
    const int tiles = a.n_q / 64, first = 256 / a.Hq > 0 ? 256 / a.Hq : 1, readers = tiles < first ? tiles : first;
    k.ahead_rows = a.K && a.key_groups == 4 && a.n_keys > 768 ? (a.n_keys + readers - 1) / readers : 0;
    const int kg = a.key_groups, waves = kg > 1 || sweep_waves(a.n_q, a.Hq) == 8 ? 8 : 4;
#define FWD_LAUNCH(D_)                                                                              \
    do {                                                                                            \
        const dim3 grid((unsigned)((a.n_q / (waves * 32 / kg)) * a.Hq));                            \
        if (kg == 4 && a.K) fwd_sweep_kernel<D_, 4, 8, true><<<grid, 512, 0, st>>>(k);              \
        else if (kg == 4) fwd_sweep_kernel<D_, 4, 8, false><<<grid, 512, 0, st>>>(k);               \
        else if (kg == 2 && a.K) fwd_sweep_kernel<D_, 2, 8, true><<<grid, 512, 0, st>>>(k);         \
        else if (kg == 2) fwd_sweep_kernel<D_, 2, 8, false><<<grid, 512, 0, st>>>(k);               \
        else if (waves == 8) fwd_sweep_kernel<D_, 1, 8, false><<<grid, 512, 0, st>>>(k);            \
        else fwd_sweep_kernel<D_, 1, 4, false><<<grid, 256, 0, st>>>(k);                            \
    } while (0)
    if (a.D == 128) FWD_LAUNCH(128);
    else if (a.D == 80) FWD_LAUNCH(80);
    else FWD_LAUNCH(64);
#undef FWD_LAUNCH
}

}  // namespace fpdt
