// Backward of the chunked attention on bf16 MFMA (Sec. 4.2; operand set of Sec. 3.1).
//
//   Delta = rowsum(dO * O)                                   (delta_kernel, HBM-bound)
//   p  = exp(scale q k^T - LSE), masked above the diagonal
//   dV += p^T dO,  dP = dO v^T,  dS = p (dP - Delta)
//   dK += scale dS^T q,  dQ += scale dS k
//
// Two MFMA kernels, each keeping its accumulators in registers and recomputing p:
//   bwd_dkdv_kernel_w4 : a workgroup (4 waves, one per SIMD) owns 256 keys of one KV head and
//       walks the query rows (all query heads of the group; where the key tiles are too few to fill
//       the chip, several workgroups share the walk and dkdv_sum_kernel adds their results).  Scores are computed as S = Q K^T
//       (queries are MFMA rows, keys are columns): a lane owns one key, and the
//       register-resident p and dS tiles are the B operands of dV^T += dO^T p and
//       dK^T += Q^T dS.
//   bwd_dq_kernel      : a workgroup (8 waves, two per SIMD, at most 256 registers each, so one
//       wave's exp / dS arithmetic runs under the other's MFMAs) owns 256 query rows of one head
//       and walks the keys with S^T = K Q^T (as in the forward): a lane owns one query, LSE and
//       Delta are per-lane scalars, and dS^T is the B operand of dQ^T += K^T dS^T.
// Both stream their operands global -> LDS directly through a small ring, as NAT fragments
// (fpdt_internal.h) only: an operand whose contraction runs over rows (Q^T, dO^T, K^T) is read
// out of the same LDS block with transposing loads.
#include <type_traits>

#include "fpdt_internal.h"
#include "mfma_tiles.h"
#include "pack_tile.h"

namespace fpdt {

namespace {

constexpr int NWAVE = 8;
constexpr int NTHREAD = NWAVE * 64;
constexpr float LOG2E = 1.4426950408889634f;

struct BwdKernelArgs {
    const uint16_t* Q; const uint16_t* dO; const uint16_t* K; const uint16_t* V;
    const u32x4* Qnat; const u32x4* dOnat;
    int64_t q_head_stride_blocks;
    const u32x4* Knat; const u32x4* Vnat;
    int64_t kv_head_stride_blocks;
    const float* LSE; const float* Delta; int64_t row_stat_stride;
    const float* stat2;  // dK/dV kernel: per (head, 32-row block) 32 x LSE * log2(e), then 32 x -Delta
    int64_t q_pos0, k_pos0;
    int n_q, n_k;
    int Hq, Hkv, g, flags;
    float scale, c;
    int splits, head_splits;  // dK/dV kernel: see launch_bwd_dkdv
    float* acc_dq; float* acc_dk; float* acc_dv;
    float* part;              // partial dK | dV of splits 1, 2, .. (splits > 1)
    uint16_t* dQ; uint16_t* dK; uint16_t* dV;
    u32x4* dS;  // dS fragments of the launch (stored-dS backward), or null
};

// Store a transposed accumulator tile set (lane = one row, registers = channels) as bf16
// into a [rows, H, D] tensor.
template <int D, int DB>
__device__ __forceinline__ void store_rows_bf16(const floatx16 (&acc)[DB], float mul, uint16_t* rowp, int half)
{
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
            const int d = 32 * db + 8 * a4 + 4 * half;
            if (d < D) {
                floatx4 v;
#pragma unroll
                for (int b = 0; b < 4; ++b) v[b] = acc[db][4 * a4 + b] * mul;
                *reinterpret_cast<bf16x4*>(rowp + d) = __builtin_convertvector(v, bf16x4);
            }
        }
}

// ---------------------------------------------------------------------------------------
// dK, dV.  Wave w owns keys [k0 + 64 w, +64) (one wave per SIMD, 4 waves, 256 keys per
// workgroup): its K fragments are stationary in registers, its V fragments are parked in LDS.
// Every step stages one 32-row query block (Q, dO, LSE * log2e, -Delta) in a 2-slot LDS ring,
// loaded one step ahead.
//
// A 32-key tile per wave needs one 1 KiB LDS fragment per MFMA, which LDS cannot deliver at
// the MFMA rate; 64 keys per wave use every Q / dO fragment twice.  The dK/dV accumulator
// registers (256 at D = 128) then have to live in AGPRs while the short-lived S / dP tiles must stay in
// architectural VGPRs (VALU cannot read AGPRs): the compiler picks one form for all MFMAs of
// a function, so the MFMAs are issued through inline assembly with explicit register classes,
// and the wait states between an MFMA result and its first VALU reader, which the compiler
// inserts for the builtin, are inserted by hand (s_nop).  The step is written in the order
// it should issue: S chains | dP chains with the exp arithmetic in their shadow | dV MFMAs
// with the dS arithmetic in their shadow | dK MFMAs.
#define FPDT_MFMA_V0(d, a, b) \
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b))
#define FPDT_MFMA_VC(d, a, b, c) \
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "v"(b), "v"(c))
#define FPDT_MFMA_V(d, a, b) \
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b))
#define FPDT_MFMA_A(d, a, b) \
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b))
// >= 11 wait states between an 8-pass MFMA writing a VGPR and a VALU instruction reading it
#define FPDT_MFMA_TO_VALU_NOPS() asm volatile("s_nop 7\n\ts_nop 4" ::: "memory")
#define FPDT_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// STORE_DS: the rounded dS tiles, which are this kernel's own MFMA operands, are also written to
// p.dS as 1 KiB fragments [head][32-query block][32-key block][s2][lane][8]: lane (key c, h') of
// fragment s2 holds dS[q = 16 s2 + 8 (e / 4) + 4 h' + e % 4][key c], e = 0..7 -- exactly the register
// contents.  bwd_dq_ds_kernel reads them back instead of recomputing S and dP.
template <int D, bool STORE_DS>
__global__ __launch_bounds__(256) void bwd_dkdv_kernel_w4(BwdKernelArgs p)
{
    constexpr int NW = 4, NK = 2;
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int NAT_U4 = DT * 64;
    constexpr int SLOT_U4 = 2 * NAT_U4;  // Q block | dO block, each once (see "Operand layout" below)
    constexpr int NFRAG = 2 * DT;
    constexpr int RING = 2;
    constexpr int BKT = NW * 32 * NK;  // keys per workgroup
    static_assert(RING == 2, "the step loops below alternate between two slots");
    // (DP > D: the transposing loads of the padded channels reach one fragment past a block;
    // the values land in accumulator columns that are never stored, the pad keeps them in LDS)
    constexpr int SLOT_PAD = DP > D ? 64 : 0;
    constexpr int UFRAG = 2 * DT + 4 * DB;  // A-operand fragments a step consumes
    constexpr int NCOPY = (NFRAG + NW - 1) / NW;
    __shared__ u32x4 slot0[SLOT_U4 + SLOT_PAD], slot1[SLOT_U4 + SLOT_PAD];
    __shared__ u32x4 vst[NW * NK * DT * 64];  // V NAT fragments of the workgroup's keys
    __shared__ __attribute__((aligned(16))) float stat0[64], stat1[64];  // LSE*log2e | -Delta

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int half = lane >> 5, col = lane & 31;
    // Split sp of a key tile takes every rsplit-th 32-row query block (rsub is the first) and g of the
    // group's heads, starting at head0.  All key tiles of one split walk the same blocks in the same
    // order, whatever the diagonal cuts off, so the splits keep the L2 sharing of the unsplit walk.
    const int kvh = blockIdx.x % p.Hkv;
    const int sp = (int)(blockIdx.x / p.Hkv) % p.splits;
    const int kt = (int)(blockIdx.x / p.Hkv) / p.splits;
    const int g = p.g / p.head_splits, rsplit = p.splits / p.head_splits, rsub = sp / p.head_splits;
    const int head0 = kvh * p.g + (sp % p.head_splits) * g;
    const int k0 = kt * BKT, kw0 = k0 + 32 * NK * wu;
    const int64_t kpos_w0 = p.k_pos0 + kw0;

    floatx16 dk[NK][DB], dv[NK][DB];
    const size_t wg = (size_t)kt * p.Hkv + kvh, n_wg = gridDim.x / (unsigned)p.splits;
    constexpr size_t WG_ACC = (size_t)(NW * NK * DB * 16 * 64);
    float* adk = (sp == 0 ? p.acc_dk : p.part + (size_t)(2 * (sp - 1)) * n_wg * WG_ACC) + wg * WG_ACC + (size_t)(w * NK) * (DB * 16 * 64);
    float* adv = (sp == 0 ? p.acc_dv : p.part + (size_t)(2 * sp - 1) * n_wg * WG_ACC) + wg * WG_ACC + (size_t)(w * NK) * (DB * 16 * 64);
    if ((p.flags & ACC_LOAD) && sp == 0) {
#pragma unroll
        for (int kb = 0; kb < NK; ++kb)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    dk[kb][db][r] = adk[((kb * DB + db) * 16 + r) * 64 + lane];
                    dv[kb][db][r] = adv[((kb * DB + db) * 16 + r) * 64 + lane];
                }
                // into accumulation registers right away, one tile pair at a time: left to the
                // first MFMA that uses them, all 256 values would sit in architectural registers
                asm volatile("" : "+a"(dk[kb][db]), "+a"(dv[kb][db]));
            }
    } else {
#pragma unroll
        for (int kb = 0; kb < NK; ++kb)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
#pragma unroll
                for (int r = 0; r < 16; ++r) dk[kb][db][r] = dv[kb][db][r] = 0.f;
                asm volatile("" : "+a"(dk[kb][db]), "+a"(dv[kb][db]));
            }
    }

    // loaded after the accumulators so that nothing has to be parked in scratch across their
    // initialisation (a reload in front of the loop would put a full vector-memory wait, which
    // also covers the operand copies in flight, at its first use inside the loop)
    bf16x8 kf[NK][DT];
    u32x4* vmine = vst + wu * (NK * DT * 64);
#pragma unroll
    for (int kb = 0; kb < NK; ++kb) {
        const size_t off = ((size_t)(kw0 + 32 * kb + col) * p.Hkv + kvh) * D + 8 * half;
        const u32x4* vsrc = p.Vnat + ((size_t)kvh * p.kv_head_stride_blocks + (kw0 / 32 + kb)) * NAT_U4;
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            kf[kb][t] = as_bf16x8(*reinterpret_cast<const u32x4*>(p.K + off + 16 * t));
            frag_to_lds(vsrc + t * 64, vmine + (kb * DT + t) * 64, lane);
        }
    }

    const int64_t qmin = p.k_pos0 + k0 - p.q_pos0;
    const int qb_start = qmin > 0 ? (int)(qmin / 32) : 0;
    const int n_qb_all = p.n_q / 32;
    const int qb_top = n_qb_all - 1 - rsub;  // the split's first block of the descending walk
    const int n_qb = qb_top >= qb_start ? (qb_top - qb_start) / rsplit + 1 : 0;
    const int n_iter = n_qb * g;
    // blocks whose first query precedes the workgroup's last key need the mask (for some wave)
    const int64_t kpos_last = p.k_pos0 + k0 + BKT - 1;
    int64_t dend = (kpos_last - p.q_pos0 + 31) / 32;
    if (dend < qb_start) dend = qb_start;
    if (dend > n_qb_all) dend = n_qb_all;
    const int n_hot_iter = qb_top >= (int)dend ? ((qb_top - (int)dend) / rsplit + 1) * g : 0;  // walked first (descending order)

    // Operand layout.  A step needs the 32 x D Q and dO blocks twice: as A operands contracted
    // over d (S = Q K^T, dP = dO V^T; lane = query row, 8 consecutive d) and contracted over the
    // query (dV^T += dO^T P, dK^T += Q^T dS; lane = d, 8 queries).  LDS holds each block ONCE, in
    // the first form's fragment order; the second form is read with the transposing LDS load
    // (ds_read_b64_tr_b16: each 16-lane group reads a 4-row x 16-column block of 16-bit values,
    // lane i of the group supplying the address of row i / 4, columns 4 (i % 4) .. +3, and lane j
    // receiving column j of the four rows).  That halves the copies and the LDS footprint of a
    // step.  Within fragment t (16 columns of d) the 16-byte piece (h', q) = row q, columns
    // 16 t + 8 h' .. +7 sits at position 32 h' + (q ^ 4 h' ^ 8 (t % 2)) instead of 32 h' + q: with
    // that swizzle the 32 lanes a transposing load serves per cycle hit 32 different 8-byte bank
    // pairs, and a plain fragment read is still a permutation of one contiguous KiB.
    //
    // Wave w copies fragments w, w+4, ... of the 2 D/16 that make a step (fragment f belongs to
    // operand f / (D/16); at D = 128 its parity is w's and its operand is known at compile time).
    // The copy engine writes lane l's 16 bytes at position l, so lane l fetches the piece that
    // belongs there.  The copies of a wave are NOT issued back
    // to back: the CU's address unit takes them one at a time, and a wave whose copy is not
    // accepted yet cannot issue its next MFMA either.  issue_begin() sets up the addresses (and
    // requests the row statistics), issue_one() sends one copy; a step calls it between its first
    // MFMA groups.
    uint64_t cp_src[2] = {0, 0};  // scalar registers: this wave's first fragment of each operand
    uint64_t stat_src = 0;
    uint64_t ds_next = 0;  // (STORE_DS) where the step that issue_begin() was last called for stores its dS fragments
    const unsigned stat_addr[2] = {lds_address(stat0), lds_address(stat1)};
    // (DT even: the parity of every fragment a wave copies is the wave's; DT odd: chosen per copy)
    const int cp_lane_par[2] = {16 * (32 * half + (col ^ (4 * half))), 16 * (32 * half + (col ^ (4 * half) ^ 8))};
    const int cp_lane_off = cp_lane_par[wu & 1];
    const unsigned slot_addr[2] = {lds_address(slot0), lds_address(slot1)};
    const unsigned slot_lds[2] = {slot_addr[0] + 1024u * (unsigned)wu, slot_addr[1] + 1024u * (unsigned)wu};
    // positions of this lane's piece in an even / odd fragment (plain fragment reads)
    const int natpos[2] = {32 * half + (col ^ (4 * half)), 32 * half + (col ^ (4 * half) ^ 8)};
    // byte offsets of this lane's two transposing loads within a block (first / second group of
    // four queries), to which 2048 db + 256 s2 is added for the fragment (32 db + .. d, 16 s2 + .. q)
    int trb[2];
    {
        const int grp = lane >> 4, i16 = lane & 15, e = i16 >> 2, x = i16 & 3;
        const int h = grp >> 1, dblk = grp & 1, hq = x >> 1;
#pragma unroll
        for (int I = 0; I < 2; ++I)
            trb[I] = 1024 * dblk + 512 * hq + 16 * (e + 4 * (h ^ hq) + 8 * (I ^ dblk)) + 8 * (x & 1);
    }
    // issue_begin(it) sets the scalar source addresses of step `it`: block (head, qb) with
    // hh = it % g, qb = qb_top - rsplit (it / g), head = head0 + hh.  It is called for it = 0, 1, 2, ..
    // in order (and once more for the last step), so the addresses are advanced by one of two
    // precomputed strides instead of being rebuilt: no division, no vector instruction, a dozen
    // scalar instructions at the head of a step, where nothing hides them.
    const int w64 = DT == 8 ? wu * 64 : 0;  // D = 128: the wave's first fragment of each operand
    const int64_t blk_next_head = p.q_head_stride_blocks;                          // hh + 1, same qb
    const int64_t blk_next_qb = -(int64_t)(g - 1) * p.q_head_stride_blocks - rsplit;  // hh wraps to 0, qb - rsplit
    const int64_t pair_next_head = (int64_t)n_qb_all * (p.n_k / 32);
    const int64_t pair_next_qb = -(int64_t)(g - 1) * pair_next_head - (int64_t)rsplit * (p.n_k / 32);
    int st_it = 0, st_hh = 0;  // the step the addresses below belong to, and its head within the group
    {
        const int64_t blk0 = (int64_t)head0 * p.q_head_stride_blocks + qb_top;
        cp_src[0] = (uint64_t)(uintptr_t)(p.Qnat + blk0 * NAT_U4 + w64);
        cp_src[1] = (uint64_t)(uintptr_t)(p.dOnat + blk0 * NAT_U4 + w64);
        stat_src = (uint64_t)(uintptr_t)(p.stat2 + blk0 * 64);
        if constexpr (STORE_DS) {
            // fragment pairs (head, query block, key block) of a launch are fewer than 2^31 (API layer)
            const int64_t pair0 = ((int64_t)head0 * n_qb_all + qb_top) * (p.n_k / 32) + kw0 / 32;
            ds_next = (uint64_t)(uintptr_t)p.dS + ((uint64_t)pair0 << 11);
        }
    }
    auto issue_begin = [&](int it) {
        if (it == st_it) return;  // the first step, and the last step's second request
        st_it = it;
        const bool wrap = ++st_hh == g;
        if (wrap) st_hh = 0;
        const int64_t db = wrap ? blk_next_qb : blk_next_head;
        cp_src[0] += (uint64_t)(db * (int64_t)(NAT_U4 * 16));
        cp_src[1] += (uint64_t)(db * (int64_t)(NAT_U4 * 16));
        // the block's row statistics (256 bytes, already in the form the step consumes) travel
        // through the copy engine like the operands: no vector register, no wait of the compiler's
        stat_src += (uint64_t)(db * 256);
        if constexpr (STORE_DS) ds_next += (uint64_t)((wrap ? pair_next_qb : pair_next_head) * 2048);
    };
    // k = 0..3 (compile-time after unrolling): fragment 4 k + w of the step, i.e. fragment
    // 4 (k % 2) + w of operand k / 2; into_slot1 is a compile-time constant at every call
    auto issue_one = [&](int k, bool into_slot1) {
        if (k == 0 && wu == 0) dwords_to_lds_at(stat_src, stat_addr[into_slot1], lane * 4);
        if constexpr (DT == 8) {
            frag_to_lds_at(cp_src[k / 2] + 1024u * (unsigned)(NW * (k % 2)), slot_lds[into_slot1] + 1024u * (unsigned)(NW * k), cp_lane_off);
        } else {
            // fragment f of the step (operand f / DT, its fragment f % DT); a wave without a
            // fragment in the last round copies its previous one again (same bytes, same place)
            int f = NW * k + wu;
            if (f >= NFRAG) f -= NW;
            const int op = f >= DT ? 1 : 0, t = f - op * DT;
            const uint64_t src = (op ? cp_src[1] : cp_src[0]) + 1024u * (unsigned)t;
            frag_to_lds_at(src, slot_addr[into_slot1] + 1024u * (unsigned)f, cp_lane_par[0] ^ (128 * (t & 1)));
        }
    };
    auto issue = [&](int it, bool into_slot1) {
        issue_begin(it);
#pragma unroll
        for (int k = 0; k < NCOPY; ++k) issue_one(k, into_slot1);
    };

    // One step.  The 32 A-operand fragments are consumed in the order Q 0..7, dO 0..7 (plain),
    // dO^T 0..7, Q^T 0..7 (transposing loads); they are read from LDS four MFMA pairs ahead into
    // a ring of six registers sets, so that a set is overwritten only two pairs after its last
    // reader was issued.
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
    auto step = [&](auto masked_tag, int it, const u32x4* sl, const float* st, u32x4* nslot, float* nst) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        (void)nst;  // filled by the copy that issue_one(0, ..) sends with the next step's operands
        const uint64_t ds_dst = ds_next;  // set when this step's operands were requested
        const bool more = it + 1 < n_iter;
        // the last step copies its own operands once more into the idle slot: the copies in the
        // MFMA sequence below then need no branch around them
        issue_begin(more ? it + 1 : it);
        if (MASKED) {  // diagonal steps (few): a wave may skip the arithmetic, so all copies go first
#pragma unroll
            for (int k = 0; k < NCOPY; ++k) issue_one(k, nslot == slot1);
        }
        const int qb = qb_top - rsplit * (it / g);
        const int64_t qpos_b0 = p.q_pos0 + (int64_t)qb * 32;

        if (!MASKED || qpos_b0 + 31 >= kpos_w0) {  // wave-uniform
            const unsigned sl_addr = slot_addr[sl == slot1];
            const unsigned tr0 = sl_addr + (unsigned)trb[0], tr1 = sl_addr + (unsigned)trb[1];
            // fragment u of the stream: 0..15 plain (Q | dO), 16..23 dO^T, 24..31 Q^T
            auto afrag = [&](int u) -> bf16x8 {
                if (u < 2 * DT) return as_bf16x8(sl[u * 64 + natpos[(u % DT) & 1]]);
                const bool of_dO = u < 2 * DT + 2 * DB;
                const int i = of_dO ? u - 2 * DT : u - 2 * DT - 2 * DB;
                const unsigned o = (of_dO ? 1024u * DT : 0u) + 2048u * (unsigned)(i % DB) + 256u * (unsigned)(i / DB);
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(tr0 + o));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(tr1 + o));
                typedef short short8v __attribute__((ext_vector_type(8)));
                const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                return __builtin_bit_cast(bf16x8, both);
            };
#define FPDT_AFRAG(u_) afrag(u_)
            // Nothing hides an LDS read that is waited for: the single wave of a SIMD stops.  At D = 64 and 80, whose pairs of MFMAs are the
            // fewest per vector instruction, V is read two pairs ahead, the statistics one chunk (both were read where they are used,
            // V one pair ahead: 32K tokens, 8 / 2 heads, D = 64 2319 -> 2102 us, 64K, 4 heads, D = 80 5433 -> 5180; at D = 128 V
            // two pairs ahead takes 0.7% longer).  Not kept: the dK MFMAs behind the next step's S, with half of the exponentials
            // between them (three slots): D = 64 another 2%, D = 80 the same, D = 128 1% longer.
            constexpr int VAHEAD = D == 128 ? 1 : 2;
            bf16x8 fr[6], vb0[3], vb1[3];
#pragma unroll
            for (int u = 0; u < 4; ++u) fr[u] = FPDT_AFRAG(u);
#pragma unroll
            for (int t = 0; t < VAHEAD; ++t) {
                vb0[t] = as_bf16x8(vmine[(0 * DT + t) * 64 + lane]);
                vb1[t] = as_bf16x8(vmine[(1 * DT + t) * 64 + lane]);
            }
            floatx16 s0, s1, dp0, dp1;
            bf16x8 pf[NK][2], df[NK][2];
            // per-row statistics are read one chunk ahead of their use and BEFORE the fragment
            // reads of that chunk, so the wait in front of the arithmetic never includes a
            // 1 KiB fragment read (LDS returns in order)
            auto stat2 = [&](int base, int r) {  // rows r, r+1 (r even): consecutive floats
                return *reinterpret_cast<const float2*>(st + base + 8 * (r >> 2) + 4 * half + (r & 3));
            };
            // The dP chains start from the tile of -Delta instead of zero (registers 4a .. 4a+3
            // hold rows 8a + 4 half + 0..3: four 16-byte reads), so the MFMAs deliver dP - Delta
            // and the dS arithmetic loses its subtraction.
            floatx16 nd;
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
                const floatx4 q4 = *reinterpret_cast<const floatx4*>(st + 32 + 8 * a4 + 4 * half);
#pragma unroll
                for (int b = 0; b < 4; ++b) nd[4 * a4 + b] = q4[b];
            }
            float2 lse[8];  // of rows 2 k, 2 k + 1 (two or three of them live at a time)
            lse[0] = stat2(0, 0);
            // ---- A: S = Q K^T, two chains ----
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                const int u = t;
                if (t == 0) {
                    FPDT_MFMA_V0(s0, fr[u % 6], kf[0][t]);
                    FPDT_MFMA_V0(s1, fr[u % 6], kf[1][t]);
                } else {
                    FPDT_MFMA_V(s0, fr[u % 6], kf[0][t]);
                    FPDT_MFMA_V(s1, fr[u % 6], kf[1][t]);
                }
                fr[(u + 4) % 6] = FPDT_AFRAG(u + 4);
                if (!MASKED && t % 2 == 0 && t / 2 < NCOPY) issue_one(t / 2, nslot == slot1);  // a copy for the next step every second MFMA pair
                FPDT_SCHED_FENCE();
            }
            // ---- B: dP - Delta = dO V^T - Delta, exp of S in the shadow of the MFMAs ----
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                const int u = DT + t;
#pragma unroll
                for (int r = 16 * t / DT; r < 16 * (t + 1) / DT; ++r)  // what the rows behind this chunk's need
                    if (r % 2 == 0 && r < 14) lse[r / 2 + 1] = stat2(0, r + 2);
                if (t == 0) {
                    FPDT_MFMA_VC(dp0, fr[u % 6], vb0[t % 3], nd);
                    FPDT_MFMA_VC(dp1, fr[u % 6], vb1[t % 3], nd);
                    FPDT_MFMA_TO_VALU_NOPS();  // s0, s1 are complete and readable from here on
                } else {
                    FPDT_MFMA_V(dp0, fr[u % 6], vb0[t % 3]);
                    FPDT_MFMA_V(dp1, fr[u % 6], vb1[t % 3]);
                }
                fr[(u + 4) % 6] = FPDT_AFRAG(u + 4);
                if (t + VAHEAD < DT) {
                    vb0[(t + VAHEAD) % 3] = as_bf16x8(vmine[(0 * DT + t + VAHEAD) * 64 + lane]);
                    vb1[(t + VAHEAD) % 3] = as_bf16x8(vmine[(1 * DT + t + VAHEAD) * 64 + lane]);
                }
                FPDT_SCHED_FENCE();
#pragma unroll
                for (int r = 16 * t / DT; r < 16 * (t + 1) / DT; ++r) {
                    const float lse2 = (r & 1) ? lse[r / 2].y : lse[r / 2].x;
                    float e0 = __builtin_amdgcn_exp2f(fmaf(s0[r], p.c, -lse2));
                    float e1 = __builtin_amdgcn_exp2f(fmaf(s1[r], p.c, -lse2));
                    if (MASKED) {
                        const int64_t qp = qpos_b0 + 8 * (r >> 2) + 4 * half + (r & 3);
                        if (kpos_w0 + col > qp) e0 = 0.f;
                        if (kpos_w0 + 32 + col > qp) e1 = 0.f;
                    }
                    s0[r] = e0;
                    s1[r] = e1;
                }
                if (16 * (t + 1) / DT >= 8 && 16 * t / DT < 8) {  // rows 0..7 are final
                    pf[0][0] = pack_half<0>(s0);
                    pf[1][0] = pack_half<0>(s1);
                }
                FPDT_SCHED_FENCE();
            }
            pf[0][1] = pack_half<1>(s0);
            pf[1][1] = pack_half<1>(s1);
            FPDT_SCHED_FENCE();
            // ---- C: dV^T += dO^T p, dS = p (dP - Delta) in the shadow (dp holds dP - Delta) ----
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) {
                const int u = 2 * DT + i;
                const int s2 = i / DB, db = i % DB;
                FPDT_MFMA_A(dv[0][db], fr[u % 6], pf[0][s2]);
                FPDT_MFMA_A(dv[1][db], fr[u % 6], pf[1][s2]);
                if (i == 0) FPDT_MFMA_TO_VALU_NOPS();  // dp0, dp1 readable
                fr[(u + 4) % 6] = FPDT_AFRAG(u + 4);
                FPDT_SCHED_FENCE();
#pragma unroll
                for (int r = 16 * i / (2 * DB); r < 16 * (i + 1) / (2 * DB); ++r) {
                    dp0[r] = s0[r] * dp0[r];
                    dp1[r] = s1[r] * dp1[r];
                }
                if (16 * (i + 1) / (2 * DB) >= 8 && 16 * i / (2 * DB) < 8) {  // rows 0..7 are final
                    df[0][0] = pack_half<0>(dp0);
                    df[1][0] = pack_half<0>(dp1);
                }
                FPDT_SCHED_FENCE();
            }
            df[0][1] = pack_half<1>(dp0);
            df[1][1] = pack_half<1>(dp1);
            FPDT_SCHED_FENCE();
            // ---- D: dK^T += Q^T dS ----
            if constexpr (STORE_DS && !MASKED) {
                // In the unmasked steps (all but a few per launch) the next step's operand copies are
                // waited for HERE, in front of this step's dS stores, not at the end of the step:
                // vector-memory stores and loads complete out of order with each other, so a wait that
                // has to cover the copies would cover the stores as well, and those have been in
                // flight for a quarter of a step only.  Issued now, the stores have a whole step to
                // drain.  (Compile-time choice: a run-time condition around the closing wait makes the
                // register allocator spill the accumulators.)
                wait_vmem_at_most<0>();
            }
#pragma unroll
            for (int i = 0; i < 2 * DB; ++i) {
                const int u = 2 * DT + 2 * DB + i;
                const int s2 = i / DB, db = i % DB;
                FPDT_MFMA_A(dk[0][db], fr[u % 6], df[0][s2]);
                FPDT_MFMA_A(dk[1][db], fr[u % 6], df[1][s2]);
                if (u + 4 < UFRAG) fr[(u + 4) % 6] = FPDT_AFRAG(u + 4);
                if constexpr (STORE_DS) {
                    // four 1 KiB stores spread over the MFMA pairs of this phase (issued behind the
                    // step's last MFMA instead, in the shadow of the barrier: 265 against 260 ms):
                    // fragment (kb, s2) of this step at [.. + kb][s2]; non-temporal, they are read
                    // back once by another kernel
                    constexpr int EVERY = 2 * DB >= 8 ? 2 : 1;
                    if (i % EVERY == 0 && i / EVERY < 4) {
                        const int f = i / EVERY;
                        uint64_t addr;  // address through a scalar move: copy_address_rule in mfma_tiles.h
                        asm volatile("s_mov_b64 %0, %3\n\tglobal_store_dwordx4 %1, %2, %0 nt"
                                     : "=&s"(addr)
                                     : "v"(lane * 16), "v"(__builtin_bit_cast(u32x4, df[f / 2][f % 2])),
                                       "s"(ds_dst + 1024u * (unsigned)f)
                                     : "memory");
                    }
                }
                FPDT_SCHED_FENCE();
            }
#undef FPDT_AFRAG
        }
        if constexpr (!STORE_DS || MASKED) wait_vmem_at_most<0>();  // the direct-to-LDS loads of step it+1 have landed
        barrier_no_fence();
    };

    if (n_iter > 0) issue(0, false);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    // Touch the stationary K fragments in front of each loop: whatever the register allocator
    // parked in scratch is reloaded and waited for HERE; a reload whose first use is inside the
    // loop would put a full vector-memory wait (operand copies in flight included) in every step.
    auto pin_kf = [&]() {
#pragma unroll
        for (int kb = 0; kb < NK; ++kb)
#pragma unroll
            for (int t = 0; t < DT; ++t) asm volatile("" ::"v"(kf[kb][t]));
    };
    // the unmasked steps come first (descending walk); an odd count leaves the ring on slot 1
    const int n_hot_even = n_hot_iter & ~1;
    pin_kf();
    for (int it = 0; it < n_hot_even; it += 2) {
        step(std::false_type{}, it, slot0, stat0, slot1, stat1);
        step(std::false_type{}, it + 1, slot1, stat1, slot0, stat0);
    }
    pin_kf();
    for (int it = n_hot_even; it < n_iter; it += 2) {
        step(std::true_type{}, it, slot0, stat0, slot1, stat1);
        if (it + 1 < n_iter) step(std::true_type{}, it + 1, slot1, stat1, slot0, stat0);
    }

    // the accumulators are read by ordinary instructions from here on
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
    if ((p.flags & ACC_FINAL) && p.splits == 1) {
#pragma unroll
        for (int kb = 0; kb < NK; ++kb) {
            const size_t off = ((size_t)(kw0 + 32 * kb + col) * p.Hkv + kvh) * D;
            store_rows_bf16<D, DB>(dk[kb], p.scale, p.dK + off, half);
            store_rows_bf16<D, DB>(dv[kb], 1.f, p.dV + off, half);
        }
    } else {
#pragma unroll
        for (int kb = 0; kb < NK; ++kb)
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    adk[((kb * DB + db) * 16 + r) * 64 + lane] = dk[kb][db][r];
                    adv[((kb * DB + db) * 16 + r) * 64 + lane] = dv[kb][db][r];
                }
    }
}

// Sum of the splits of a dK/dV launch: acc += partials, or, with ACC_FINAL, the rounded outputs.  One
// wave per 32-key x 32-channel accumulator tile; blockIdx.y = 0: dK, 1: dV.  Memory-bound: (splits + 1)
// passes over n_k * Hkv * D fp32 values each of dK and dV.
template <int D>
__global__ __launch_bounds__(256) void dkdv_sum_kernel(BwdKernelArgs p, unsigned n_wg)
{
    constexpr int NW = 4, NK = 2, DB = (D + 31) / 32;
    constexpr int TILE = 16 * 64;
    const unsigned lane = threadIdx.x & 63;
    const size_t tile = (size_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (workgroup, wave, key block, channel block)
    const bool is_v = blockIdx.y != 0;
    const size_t all = (size_t)n_wg * (NW * NK * DB) * TILE;  // floats per operand
    float* acc = (is_v ? p.acc_dv : p.acc_dk) + tile * TILE + lane;
    const float* part = p.part + (is_v ? all : 0) + tile * TILE + lane;
    floatx16 v;
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = acc[r * 64];
    for (int sp = 1; sp < p.splits; ++sp, part += 2 * all) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] += part[r * 64];
    }
    if (!(p.flags & ACC_FINAL)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r * 64] = v[r];
        return;
    }
    const int half = (int)lane >> 5, col = (int)lane & 31;
    const unsigned db = (unsigned)(tile % DB), blk = (unsigned)(tile / DB) % (NW * NK), wg = (unsigned)(tile / (DB * NW * NK));
    const size_t key = (size_t)(wg / (unsigned)p.Hkv) * (NW * NK * 32) + 32 * blk + col;
    uint16_t* row = (is_v ? p.dV : p.dK) + (key * p.Hkv + wg % (unsigned)p.Hkv) * D;
    const float mul = is_v ? 1.f : p.scale;
#pragma unroll
    for (int a4 = 0; a4 < 4; ++a4) {
        const int d = 32 * (int)db + 8 * a4 + 4 * half;
        if (d < D) {
            floatx4 o;
#pragma unroll
            for (int b = 0; b < 4; ++b) o[b] = v[4 * a4 + b] * mul;
            *reinterpret_cast<bf16x4*>(row + d) = __builtin_convertvector(o, bf16x4);
        }
    }
}

// ---------------------------------------------------------------------------------------
// dQ.  Wave w owns query rows [q0 + 32 w, +32) of one head (Q and dO fragments, LSE and Delta
// stationary in registers).  Every step stages a 64-key tile (K-NAT, V-NAT, K-TR) in a 3-slot
// LDS ring, loaded two tiles ahead.
//
// What bounds it is how well the vector work of a block hides under MFMAs, and the instructions of a wave, of which two on a SIMD issue
// one in about five clocks each: exponentials stand between the MFMAs of dP, the second half of dS between those of dQ, positions are
// 32-bit, a copy takes five instructions.  us, vector work behind the MFMAs it follows -> this (8 / 2 heads, D = 128; 64 last): 2K
// 32.2 -> 30.1, 8K 195 -> 189, 64K 10504 -> 10159 (1300 TFLOP/s executed); 64K 6020 -> 5761.
//
// KG = 2, 4 (as in the forward): 128 or 64 query rows per workgroup, the waves of one row block take every
// KG-th 32-key block and add their results through LDS at the end (dq_key_groups).
template <int D, int KG>
__global__ __launch_bounds__(NTHREAD) void bwd_dq_kernel(BwdKernelArgs p)
{
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int KB = KG == 1 ? 2 : 1;                // 32-key blocks of a wave per tile
    constexpr int NB = KG * KB, BK = NB * 32;          // blocks and keys per tile
    constexpr int NQ = NWAVE / KG, BQ = NQ * 32;
    constexpr int NAT_U4 = NB * DT * 64;  // per tile of BK keys
    // The K tile is staged once; the key-contracted operand of dQ^T += K^T dS^T is read from the
    // same block with transposing LDS loads (layout and swizzle as in the dK/dV kernel above,
    // keys in the place of queries).  With DP > D the loads of the padded channels reach into the
    // next fragments of the slot; they only feed accumulator columns that are never stored.
    constexpr int SLOT_U4 = 2 * NAT_U4;
    constexpr int NATF = NB * DT, NFRAG = 2 * NATF;
    constexpr int RING = KG == 4 ? 2 : 3, PF = RING - 1;
    // (DP > D: the transposing loads of the last block's padded channels stay within its slot: V follows K)
    __shared__ u32x4 ring_a[KG == 1 ? SLOT_U4 : RING * SLOT_U4], ring_b[KG == 1 ? SLOT_U4 : 1], ring_c[KG == 1 ? SLOT_U4 : 1];
    u32x4* const ring0 = ring_a;
    u32x4* const ring1 = KG == 1 ? ring_b : ring_a + SLOT_U4;
    u32x4* const ring2 = KG == 1 ? ring_c : ring_a + (RING - 1) * SLOT_U4;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int half = lane >> 5, col = lane & 31;
    const int qb = KG == 1 ? w : wu % NQ, kg = KG == 1 ? 0 : wu / NQ;  // this wave's row block and its share of the key blocks
    const int head = blockIdx.x % p.Hq;
    const int n_qt = p.n_q / BQ;
    const int qt = n_qt - 1 - (int)(blockIdx.x / p.Hq);
    const int kvh = head / p.g;
    const int q0 = qt * BQ, qw0 = q0 + qb * 32;

    const int ahead_pos = (int)(p.q_pos0 - p.k_pos0) + q0;  // position of the workgroup's first row behind the launch's first key (below 2^30)
    int need = ahead_pos + BQ < p.n_k ? ahead_pos + BQ : p.n_k;
    if (need < 0) need = 0;
    const int n_tiles = (need + BK - 1) / BK;

    const int natpos[2] = {32 * half + (col ^ (4 * half)), 32 * half + (col ^ (4 * half) ^ 8)};
    int trb[2];  // byte offsets of this lane's two transposing loads within a 32-key block
    {
        const int grp = lane >> 4, i16 = lane & 15, e = i16 >> 2, x = i16 & 3;
        const int h = grp >> 1, dblk = grp & 1, hq = x >> 1;
#pragma unroll
        for (int I = 0; I < 2; ++I)
            trb[I] = 1024 * dblk + 512 * hq + 16 * (e + 4 * (h ^ hq) + 8 * (I ^ dblk)) + 8 * (x & 1);
    }
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef short short8v __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
    // This wave's copies of a tile: fragments w, w + 8, .. of K and of V.  (A wave without one in the last round copies another's once more: at D
    // = 80 32 copies for 20 fragments with one key group.)
    constexpr int COPIES = (NATF + NWAVE - 1) / NWAVE;
    static_assert(COPIES * NWAVE <= 2 * NATF, "every wave has something to copy");
    unsigned cp_at[COPIES], k_off[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
        const int f = NWAVE * i + wu < NATF ? NWAVE * i + wu : NWAVE * i + wu - NATF;
        cp_at[i] = 1024u * (unsigned)f;
        // a K fragment's 16-byte pieces land swizzled by the parity of its index within the key block (DT even: that is the wave's parity)
        k_off[i] = 16u * (unsigned)((32 * half + (col ^ (4 * half))) ^ (8 * ((DT % 2 == 0 ? wu : f % DT) & 1)));
    }
    uint64_t k_src = uniform((uint64_t)(uintptr_t)(p.Knat + (size_t)kvh * p.kv_head_stride_blocks * (DT * 64)));
    uint64_t v_src = uniform((uint64_t)(uintptr_t)(p.Vnat + (size_t)kvh * p.kv_head_stride_blocks * (DT * 64)));
    auto issue = [&](const u32x4* slot) {  // the tile that comes next
        const unsigned lds = lds_address(slot);
#pragma unroll
        for (int i = 0; i < COPIES; ++i) copy_1k(k_src + cp_at[i], lds, cp_at[i], k_off[i]);
#pragma unroll
        for (int i = 0; i < COPIES; ++i) copy_1k(v_src + cp_at[i], lds + 16u * NAT_U4, cp_at[i], 16u * (unsigned)lane);
        k_src += NAT_U4 * 16;
        v_src += NAT_U4 * 16;
    };

    bf16x8 qf[DT], of[DT];
    const int row = qw0 + col;
    {
        const size_t off = ((size_t)row * p.Hq + head) * D + 8 * half;
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            qf[t] = as_bf16x8(*reinterpret_cast<const u32x4*>(p.Q + off + 16 * t));
            of[t] = as_bf16x8(*reinterpret_cast<const u32x4*>(p.dO + off + 16 * t));
        }
    }
    const float lse2 = p.LSE[(size_t)head * p.row_stat_stride + row] * LOG2E;
    // The dP chain starts from -Delta instead of zero, so the MFMAs deliver dP - Delta directly
    // (one vector instruction per element less; plain vector instructions take issue slots from
    // the MFMAs of the SIMD's other wave).  The same trick for the scores would need Q held
    // pre-multiplied by scale * log2(e) in bf16: measured, that rounding alone pushes dQ past its
    // error budget (the cancellation in p (dP - Delta) amplifies it), so the scores keep their
    // fp32 multiply-add.
    floatx16 neg_delta;
    {
        const float dl = -p.Delta[(size_t)head * p.row_stat_stride + row];
#pragma unroll
        for (int r = 0; r < 16; ++r) neg_delta[r] = dl;
    }

    floatx16 acc[DB];
    // accumulator slot of the row block: the same whatever KG a launch of the call has
    float* aq = p.acc_dq + ((size_t)(qw0 / 32) * p.Hq + head) * (size_t)(DB * 16 * 64);
    if ((p.flags & ACC_LOAD) && kg == 0) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = aq[(db * 16 + r) * 64 + lane];
    } else {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    }

    if (n_tiles > 0) issue(ring0);
    if (PF > 1 && n_tiles > 1) issue(ring1);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    const int reach = ahead_pos + 32 * qb;         // of the wave's first row behind the launch's first key
    const int row_key = reach + col - 4 * half;    // the last key this lane's query sees, less the lane's offset
    const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // One tile: compute on slot `kn`, prefetch tile it+PF into slot `pf_slot`.  A block is straight code in three steps, whose vector work stands
    // between MFMAs that do not depend on it: S, with the reads of V | dP with exp(S) and the reads of K^T | dQ with the second half of dS.
    auto tile = [&](int it, const u32x4* kn, u32x4* pf_slot) {
        if (it + PF < n_tiles) issue(pf_slot);
        const u32x4* vn = kn + NAT_U4;
        const unsigned kn_addr = lds_address(kn);
#pragma unroll
        for (int kb_i = 0; kb_i < KB; ++kb_i) {
            const int kb = kg * KB + kb_i;
            const int key0 = it * BK + 32 * kb;
            if (key0 <= reach + 31) {  // wave-uniform
                bf16x8 kfr[DT], vfr[DT], tfr[2][DB];
#pragma unroll
                for (int t = 0; t < DT; ++t) kfr[t] = as_bf16x8(kn[(kb * DT + t) * 64 + natpos[t & 1]]);
                floatx16 s, dp;
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    s = mfma32(kfr[t], qf[t], t == 0 ? zero : s);
                    vfr[t] = as_bf16x8(vn[(kb * DT + t) * 64 + lane]);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, DT, 0);
#pragma unroll
                for (int t = 0; t < DT; ++t) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
                asm volatile("" ::: "memory");  // (the reads of V stay in front of the branch)
                if (key0 + 31 > reach) {  // wave-uniform: the block straddles the diagonal
                    const int last = row_key - key0;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (8 * (r >> 2) + (r & 3) > last) s[r] = -INFINITY;
                }
                for_each<DT>([&](auto step) {
                    constexpr int t = decltype(step)::value;
                    dp = mfma32(vfr[t], of[t], t == 0 ? neg_delta : dp);
#pragma unroll
                    for (int i = reads_before(t, DT, 2 * DB); i < reads_before(t + 1, DT, 2 * DB); ++i) {
                        const unsigned o = kn_addr + 1024u * (unsigned)(kb * DT) + 2048u * (unsigned)(i % DB) + 256u * (unsigned)(i / DB);
                        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(o + (unsigned)trb[0]));
                        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)(o + (unsigned)trb[1]));
                        const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                        tfr[i / DB][i % DB] = __builtin_bit_cast(bf16x8, both);
                    }
#pragma unroll
                    for (int r = 16 * t / DT; r < 16 * (t + 1) / DT; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], p.c, -lse2));
                    __builtin_amdgcn_sched_barrier(0);
                });
                bf16x8 df[2];
#pragma unroll
                for (int r = 0; r < 8; ++r) dp[r] = s[r] * dp[r];
                df[0] = pack_half<0>(dp);
                for_each<2 * DB>([&](auto step) {
                    constexpr int i = decltype(step)::value;
                    acc[i % DB] = mfma32(tfr[i / DB][i % DB], df[i / DB], acc[i % DB]);
#pragma unroll
                    for (int r = 8 + 8 * i / DB; i < DB && r < 8 + 8 * (i + 1) / DB; ++r) dp[r] = s[r] * dp[r];
                    if (i == DB - 1) df[1] = pack_half<1>(dp);
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
        }
        // tile it+1 must have landed; the loads of tile it+PF issued above may stay in flight (PF = 2)
        if (it + PF < n_tiles) wait_vmem_at_most<(PF - 1) * 2 * COPIES>();
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

    // The lane's number once more, and what follows from it: kept through the loop, at D = 128 with several key groups, three registers of
    // it would go to scratch memory.
    const int end_lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)), end_row = qw0 + (end_lane & 31);
    if constexpr (KG > 1) {  // (the loop ended with a barrier behind the last reads of the ring)
        constexpr int PART = DB * 16 * 64;
        static_assert((NWAVE - NQ) * PART * 4 <= RING * SLOT_U4 * 16, "the ring holds the parts");
        __syncthreads();
        float* part = reinterpret_cast<float*>(ring_a);
        if (kg > 0) {
            float* mine = part + (size_t)((kg - 1) * NQ + qb) * PART + end_lane;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) mine[(db * 16 + r) * 64] = acc[db][r];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int i = 1; i < KG; ++i) {
            const float* other = part + (size_t)((i - 1) * NQ + qb) * PART + end_lane;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] += other[(db * 16 + r) * 64];
        }
    }

    if (p.flags & ACC_FINAL) {
        store_rows_bf16<D, DB>(acc, p.scale, p.dQ + ((size_t)end_row * p.Hq + head) * D, end_lane >> 5);
    } else {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) aq[(db * 16 + r) * 64 + end_lane] = acc[db][r];
    }
}

// ---------------------------------------------------------------------------------------
// dQ from stored dS (the stored-dS backward).  The dK/dV kernel has written the rounded dS tiles
// of the launch; dQ^T += K^T dS^T is then ONE GEMM per chunk pair instead of three (no S, no dP,
// no exp).  Per chunk pair the tiles are n_q * n_k * Hq * 2 bytes, read once from HBM, which is
// what bounds this kernel; its MFMA work is a third of bwd_dq_kernel's.
//
// Workgroup = 8 waves x 32 query rows of one head, as in bwd_dq_kernel (4 or 2 waves where a launch
// has few row tiles, sweep_waves).  Per 64-key tile the K-NAT block is staged once for all waves (same layout, swizzle and transposing loads as above)
// and every wave stages the four dS fragments (2 key blocks x 2 query halves) of ITS query block.
// A stored fragment holds, per key, eight queries; the B operand of dQ^T += K^T dS^T wants, per
// query, eight keys: the same transposing LDS load delivers that (4 keys x 16 queries per 16-lane
// group and load).  The 16-byte piece of writer lane (key c, h') of fragment s2 is placed at
// position 32 h' + (c ^ 4 h' ^ 8 s2) by the copy's per-lane source address, so that the 32 lanes
// one load serves per cycle touch 32 different 8-byte bank pairs.
template <int D, int NWAVE>
__global__ __launch_bounds__(NWAVE * 64, 2) void bwd_dq_ds_kernel(BwdKernelArgs p)
{
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int BK = 64, KB = BK / 32;
    constexpr int BQ = NWAVE * 32;
    constexpr int NATF = KB * DT;            // K fragments per tile (shared by the workgroup)
    constexpr int K_U4 = NATF * 64;
    constexpr int K_PAD = DP > D ? 64 : 0;   // transposing loads of padded channels reach past the block
    constexpr int DSF = KB * 2;              // dS fragments per tile and wave
    constexpr int DS_U4 = DSF * 64;
    constexpr int RING = 3;
    static_assert(RING == 3, "the tile loop below is unrolled over three slots");
    __shared__ u32x4 kring0[K_U4 + K_PAD], kring1[K_U4 + K_PAD], kring2[K_U4 + K_PAD];
    __shared__ u32x4 dring0[NWAVE * DS_U4], dring1[NWAVE * DS_U4], dring2[NWAVE * DS_U4];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int half = lane >> 5, col = lane & 31;
    const int head = blockIdx.x % p.Hq;
    const int n_qt = p.n_q / BQ;
    const int qt = n_qt - 1 - (int)(blockIdx.x / p.Hq);
    const int kvh = head / p.g;
    const int q0 = qt * BQ, qw0 = q0 + w * 32;

    const int64_t last_q_pos = p.q_pos0 + q0 + BQ - 1;
    int64_t need = last_q_pos - p.k_pos0 + 1;
    if (need > p.n_k) need = p.n_k;
    if (need < 0) need = 0;
    const int n_tiles = (int)((need + BK - 1) / BK);

    const u32x4* knb = p.Knat + (size_t)kvh * p.kv_head_stride_blocks * (DT * 64);
    // this wave's dS fragments: [head][query block][key block][s2][64 lanes]
    const u32x4* dsb = p.dS + (((size_t)head * (unsigned)(p.n_q / 32) + (unsigned)(q0 / 32 + wu)) * (unsigned)(p.n_k / 32)) * 128;

    const int cp_lane0 = 32 * half + (col ^ (4 * half));  // K fragments: even index within the key block; odd: ^ 8
    int trb[2];  // K^T: byte offsets of this lane's two transposing loads within a 32-key block
    int dsb_off[2];  // dS^T: the same for the wave's dS fragments of one key block
    {
        const int grp = lane >> 4, i16 = lane & 15, e = i16 >> 2, x = i16 & 3;
        const int h = grp >> 1, dblk = grp & 1, hq = x >> 1;
#pragma unroll
        for (int I = 0; I < 2; ++I)
            trb[I] = 1024 * dblk + 512 * hq + 16 * (e + 4 * (h ^ hq) + 8 * (I ^ dblk)) + 8 * (x & 1);
        // group (h, s2 = query half); lane i16 supplies row r = i16 / 4 (a key) and piece m = i16 % 4:
        // writer half h' = m % 2, upper or lower 8 bytes m / 2.  Keys of a 16-key step come in the
        // order 8 I + 4 h + r, the row order of the K^T operand above.
        const int s2 = grp & 1, r = i16 >> 2, m = i16 & 3, hw = m & 1, up = m >> 1;
#pragma unroll
        for (int I = 0; I < 2; ++I)
            dsb_off[I] = 1024 * s2 + 16 * (32 * hw + 8 * (I ^ s2) + 4 * (h ^ hw) + r) + 8 * up;
    }
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef short short8v __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
    auto tr_frag = [&](unsigned a0, unsigned a1) -> bf16x8 {
        const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)a0);
        const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(uintptr_t)a1);
        const short8v both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf16x8, both);
    };
    // source piece of this lane's LDS position in a dS fragment of query half s2
    const int ds_src[2] = {32 * half + (col ^ (4 * half)), 32 * half + (col ^ (4 * half) ^ 8)};
    auto issue = [&](int it, u32x4* kslot, u32x4* dslot) {
#pragma unroll
        for (int f0 = 0; f0 < NATF; f0 += NWAVE) {
            const int f = f0 + wu;
            if (f0 + NWAVE <= NATF || f < NATF) {
                const int par = DT % 2 == 0 ? (wu & 1) : ((f % DT) & 1);
                frag_to_lds(knb + (size_t)it * K_U4 + f * 64, kslot + f * 64, cp_lane0 ^ (8 * par));
            }
        }
        u32x4* mine = dslot + wu * DS_U4;
#pragma unroll
        for (int f = 0; f < DSF; ++f) frag_to_lds_nt(dsb + ((size_t)it * DSF + f) * 64, mine + f * 64, ds_src[f & 1]);
    };

    floatx16 acc[DB];
    const size_t wg = blockIdx.x;
    float* aq = p.acc_dq + (wg * NWAVE + w) * (size_t)(DB * 16 * 64);
    if (p.flags & ACC_LOAD) {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = aq[(db * 16 + r) * 64 + lane];
    } else {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    }

    if (n_tiles > 0) issue(0, kring0, dring0);
    if (n_tiles > 1) issue(1, kring1, dring1);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();

    const int64_t qpos_last = p.q_pos0 + qw0 + 31;
    constexpr int NCOPY = NATF / NWAVE + DSF;  // copies EVERY wave issues per tile (some issue one more)
    auto tile = [&](int it, const u32x4* kn, const u32x4* dsl, u32x4* pf_k, u32x4* pf_d) {
        if (it + 2 < n_tiles) issue(it + 2, pf_k, pf_d);
        const unsigned kn_addr = lds_address(kn);
        const unsigned ds_addr = lds_address(dsl + wu * DS_U4);
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int64_t key0 = p.k_pos0 + (int64_t)it * BK + 32 * kb;
            if (key0 <= qpos_last) {  // wave-uniform: the dK/dV kernel wrote exactly these blocks
                bf16x8 bfr[2], tfr[2][DB];
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2) {
                    const unsigned o = ds_addr + 2048u * (unsigned)kb + 256u * (unsigned)s2;
                    bfr[s2] = tr_frag(o + (unsigned)dsb_off[0], o + (unsigned)dsb_off[1]);
                }
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int db = 0; db < DB; ++db) {
                        const unsigned o = kn_addr + 16u * 64u * (unsigned)(kb * DT) + 2048u * (unsigned)db + 256u * (unsigned)s2;
                        tfr[s2][db] = tr_frag(o + (unsigned)trb[0], o + (unsigned)trb[1]);
                    }
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    acc[db] = mfma32(tfr[0][db], bfr[0], acc[db]);
                    acc[db] = mfma32(tfr[1][db], bfr[1], acc[db]);
                }
            }
        }
        if (it + 2 < n_tiles) wait_vmem_at_most<NCOPY>();
        else wait_vmem_at_most<0>();
        barrier_no_fence();
    };
    for (int it = 0; it < n_tiles; it += 3) {
        tile(it, kring0, dring0, kring2, dring2);
        if (it + 1 < n_tiles) tile(it + 1, kring1, dring1, kring0, dring0);
        if (it + 2 < n_tiles) tile(it + 2, kring2, dring2, kring1, dring1);
    }

    const int row = qw0 + col;
    if (p.flags & ACC_FINAL) {
        store_rows_bf16<D, DB>(acc, p.scale, p.dQ + ((size_t)row * p.Hq + head) * D, half);
    } else {
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) aq[(db * 16 + r) * 64 + lane] = acc[db][r];
    }
}

// ---------------------------------------------------------------------------------------
// Row statistics in the form the dK/dV kernel consumes, so that its steps can fetch them with a
// plain 256-byte copy: out[head][32-row block][0..31] = LSE * log2(e), [32..63] = -Delta.
__global__ __launch_bounds__(256) void stat_pack_kernel(const float* __restrict__ LSE, const float* __restrict__ Delta,
                                                        int64_t stride, int64_t n_blocks, int Hq,
                                                        int64_t out_head_stride_blocks, float* __restrict__ out)
{
    const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);  // (head, block) pair
    if (item >= n_blocks * Hq) return;
    const int64_t head = item / n_blocks, blk = item % n_blocks;
    const int t = threadIdx.x & 63;
    const float v = (t < 32 ? LSE : Delta - 32)[(size_t)head * stride + blk * 32 + t];
    out[((size_t)head * out_head_stride_blocks + blk) * 64 + t] = t < 32 ? v * LOG2E : -v;
}

// ---------------------------------------------------------------------------------------
// Delta[h][row] = sum_d dO * O.  16 lanes per (row, head), 16 bytes of each tensor per lane and access
// (all head dimensions are multiples of 16, the tensors 16-byte aligned).  HBM-bound: 131072 rows x 8
// heads, D = 128, bf16 97 us (5.5 TB/s; with 2-byte loads 156).
typedef float float4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float dot16(const float* a, const float* b)
{
    const float4v x = *reinterpret_cast<const float4v*>(a), y = *reinterpret_cast<const float4v*>(b);
    return fmaf(x[0], y[0], fmaf(x[1], y[1], fmaf(x[2], y[2], x[3] * y[3])));
}
__device__ __forceinline__ float dot16(const uint16_t* a, const uint16_t* b)
{
    const u32x4 x = *reinterpret_cast<const u32x4*>(a), y = *reinterpret_cast<const u32x4*>(b);
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s = fmaf(__uint_as_float(x[i] << 16), __uint_as_float(y[i] << 16), s);
        s = fmaf(__uint_as_float(x[i] & 0xffff0000u), __uint_as_float(y[i] & 0xffff0000u), s);
    }
    return s;
}

// sum_d dO * O of one row, by sixteen lanes (sub = 0..15), each of which has it
template <typename T>
__device__ __forceinline__ float delta_of_row(const T* __restrict__ o, const T* __restrict__ g, int D, int sub)
{
    constexpr int V = 16 / (int)sizeof(T);
    float acc = 0.f;
    for (int d = V * sub; d < D; d += 16 * V) acc += dot16(o + d, g + d);
#pragma unroll
    for (int m = 8; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
    return acc;
}
// One row's statistics where the dK/dV kernel reads them (stat_pack_kernel's output)
__device__ __forceinline__ void put_stats(float* stat2, int64_t head_stride_blocks, int head, int64_t row, float lse, float delta)
{
    float* at = stat2 + ((size_t)head * head_stride_blocks + row / 32) * 64 + row % 32;
    at[0] = lse * LOG2E;
    at[32] = -delta;
}

template <typename T>
__global__ __launch_bounds__(256) void delta_kernel(const T* __restrict__ O, const T* __restrict__ dO,
                                                    int64_t rows, int Hq, int D, float* __restrict__ Delta,
                                                    int64_t stride, unsigned* __restrict__ clear, int n_clear)
{
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_clear; i += 256) clear[i] = 0;
    // 16 lanes per (row, head): 4 pairs per wave, 16 pairs per workgroup
    const int tid = threadIdx.x;
    const int64_t pair = (int64_t)blockIdx.x * 16 + (tid >> 4);
    const int sub = tid & 15;
    if (pair >= rows * Hq) return;  // whole 16-lane groups leave together
    const float acc = delta_of_row<T>(O + (size_t)pair * D, dO + (size_t)pair * D, D, sub);
    if (sub == 0) {
        const int64_t row = pair / Hq;
        const int h = (int)(pair % Hq);
        Delta[(size_t)h * stride + row] = acc;
    }
}


// Exact Delta for the first rows of the sequence: Delta_i = sum_j p_ij (dO_i . v_j).
// rowsum(dO * O) inherits the bf16 rounding of the stored O; for a row with only a few keys
// the softmax is often peaked, dS = p (dP - Delta) then cancels almost completely and that
// rounding dominates dQ.  Its weight decays like 1/sqrt(row), so only the head of the
// sequence is recomputed.
// One workgroup per (32-row block, head); wave w takes key block w (of at most 8) through the same
// MFMAs as the dQ kernel, straight from the row-major tensors, and the eight partial row sums meet in
// LDS.  Latency-bound: 10 us in place of the 176 us of one wave per row with a scalar dot product
// per lane and key (D = 128, 8 heads).
// stat2 (or null): what stat_pack_kernel makes of these rows, head stride stat2_blocks blocks.
template <int D>
__device__ __forceinline__ void delta_head_block(const uint16_t* __restrict__ Q, const uint16_t* __restrict__ dO, const uint16_t* __restrict__ K,
                                                 const uint16_t* __restrict__ V, const float* __restrict__ LSE, int64_t stat_stride, int Hq, int Hkv,
                                                 float c, float* __restrict__ Delta, float* __restrict__ stat2, int64_t stat2_blocks, unsigned block)
{
    constexpr int DT = D / 16;
    static_assert(DELTA_HEAD_ROWS == 256, "one wave per 32-key block");
    __shared__ float part[8][32];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, half = lane >> 5, col = lane & 31;
    const int rb = block / (unsigned)Hq, head = block % (unsigned)Hq, kvh = head / (Hq / Hkv);
    const int row = 32 * rb + col;
    float sum = 0.f;
    if (w <= rb) {
        const size_t qo = ((size_t)row * Hq + head) * D + 8 * half, ko = ((size_t)(32 * w + col) * Hkv + kvh) * D + 8 * half;
        floatx16 s = {}, dp = {};
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            s = mfma32(as_bf16x8(*reinterpret_cast<const u32x4*>(K + ko + 16 * t)), as_bf16x8(*reinterpret_cast<const u32x4*>(Q + qo + 16 * t)), s);
            dp = mfma32(as_bf16x8(*reinterpret_cast<const u32x4*>(V + ko + 16 * t)), as_bf16x8(*reinterpret_cast<const u32x4*>(dO + qo + 16 * t)), dp);
        }
        const float lse2 = LSE[(size_t)head * stat_stride + row] * LOG2E;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (32 * w + acc_row(r, lane) <= row) sum = fmaf(__builtin_amdgcn_exp2f(fmaf(s[r], c, -lse2)), dp[r], sum);
        sum += xor32(sum);
    }
    if (half == 0) part[w][col] = sum;
    __syncthreads();
    if (threadIdx.x < 32) {
        float total = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) total += part[i][threadIdx.x];
        Delta[(size_t)head * stat_stride + 32 * rb + threadIdx.x] = total;
        if (stat2) put_stats(stat2, stat2_blocks, head, 32 * rb + threadIdx.x, LSE[(size_t)head * stat_stride + 32 * rb + threadIdx.x], total);
    }
}
template <int D>
__global__ __launch_bounds__(512) void delta_head_kernel(const uint16_t* __restrict__ Q,
                                                         const uint16_t* __restrict__ dO,
                                                         const uint16_t* __restrict__ K,
                                                         const uint16_t* __restrict__ V,
                                                         const float* __restrict__ LSE, int64_t stat_stride,
                                                         int Hq, int Hkv, float c, float* __restrict__ Delta)
{
    delta_head_block<D>(Q, dO, K, V, LSE, stat_stride, Hq, Hkv, c, Delta, nullptr, 0, blockIdx.x);
}

// What the two kernels of a backward over the whole sequence need, in one launch: Delta and the row statistics (the first
// DELTA_HEAD_ROWS rows from the exact sum, the others from the stored O) and the packed operands.  Workgroups of 512 threads: first those of the
// exact rows, which take longest, then one per 32-row block and head for Delta, then the packed blocks.  Four launches of 4 to 11 us with
// their gaps before: 8 / 2 heads, D = 128, backward of 2K tokens 94.1 -> 85.5 us, of 8K 471 -> 463.
struct PrepareArgs {
    const uint16_t *Q, *dO, *K, *V, *O;
    const float* LSE;
    float *Delta, *stat2;
    int64_t S;
    int Hq, Hkv;
    float c;
    PackJobs jobs;
    unsigned head_blocks, delta_blocks, first;  // first: block of the launch's first workgroup
};
template <int D>
__global__ __launch_bounds__(512) void bwd_prepare_kernel(PrepareArgs p)
{
    unsigned block = p.first + blockIdx.x;
    if (block < p.head_blocks) {
        delta_head_block<D>(p.Q, p.dO, p.K, p.V, p.LSE, p.S, p.Hq, p.Hkv, p.c, p.Delta, p.stat2, p.S / 32, block);
        return;
    }
    block -= p.head_blocks;
    if (block < p.delta_blocks) {
        const int head = block % (unsigned)p.Hq, sub = threadIdx.x & 15;
        const int64_t row = DELTA_HEAD_ROWS + (int64_t)(block / (unsigned)p.Hq) * 32 + (threadIdx.x >> 4);
        const size_t at = ((size_t)row * p.Hq + head) * D;
        const float delta = delta_of_row<uint16_t>(p.O + at, p.dO + at, D, sub);
        if (sub == 0) {
            p.Delta[(size_t)head * p.S + row] = delta;
            put_stats(p.stat2, p.S / 32, head, row, p.LSE[(size_t)head * p.S + row], delta);
        }
        return;
    }
    block -= p.delta_blocks;
    const unsigned heads = 2 * (unsigned)(p.Hq + p.Hkv);
    pack_tile<D, 512>(p.jobs, p.S / 32, block / heads, (int)(block % heads));
}

}  // namespace

int bwd_k_tile(int D) { (void)D; return NWAVE * 32; }
int bwd_q_tile(int D) { (void)D; return NWAVE * 32; }
size_t bwd_acc_dq_bytes(int64_t n_q, int Hq, int D) { return (size_t)n_q * Hq * dpad(D) * sizeof(float); }
size_t bwd_acc_dkv_bytes(int64_t n_k, int Hkv, int D) { return (size_t)n_k * Hkv * dpad(D) * sizeof(float); }

static BwdKernelArgs to_kernel_args(const BwdArgs& a)
{
    BwdKernelArgs k;
    k.Q = (const uint16_t*)a.Q; k.dO = (const uint16_t*)a.dO;
    k.K = (const uint16_t*)a.K; k.V = (const uint16_t*)a.V;
    k.Qnat = (const u32x4*)a.Qnat;
    k.dOnat = (const u32x4*)a.dOnat;
    k.q_head_stride_blocks = a.q_head_stride_blocks;
    k.Knat = (const u32x4*)a.Knat; k.Vnat = (const u32x4*)a.Vnat;
    k.kv_head_stride_blocks = a.kv_head_stride_blocks;
    k.LSE = a.LSE; k.Delta = a.Delta; k.row_stat_stride = a.row_stat_stride;
    k.stat2 = a.stat2;
    k.q_pos0 = a.q_pos0; k.k_pos0 = a.k_pos0;
    k.n_q = (int)a.n_q; k.n_k = (int)a.n_k;
    k.Hq = a.Hq; k.Hkv = a.Hkv; k.g = a.Hq / a.Hkv; k.flags = a.flags;
    k.scale = a.scale; k.c = a.scale * LOG2E;
    k.acc_dq = a.acc_dq; k.acc_dk = a.acc_dk; k.acc_dv = a.acc_dv;
    k.splits = a.dkdv_splits; k.part = a.dkdv_part;
    k.head_splits = 1;  // the largest common divisor of the splits and the group's heads
    for (int h = 2; h <= a.dkdv_splits && h <= k.g; ++h)
        if (a.dkdv_splits % h == 0 && k.g % h == 0) k.head_splits = h;
    k.dQ = (uint16_t*)a.dQ; k.dK = (uint16_t*)a.dK; k.dV = (uint16_t*)a.dV;
    k.dS = (u32x4*)a.dS_frag;
    return k;
}

size_t bwd_part_dkdv_bytes(int64_t n_k, int Hkv, int D, int splits) { return 2 * (size_t)(splits - 1) * bwd_acc_dkv_bytes(n_k, Hkv, D); }

void launch_bwd_dkdv(const BwdArgs& a, hipStream_t st)
{
    const BwdKernelArgs k = to_kernel_args(a);
    const unsigned n_wg = (unsigned)((a.n_k / bwd_k_tile(a.D)) * a.Hkv);
    dim3 grid(n_wg * (unsigned)k.splits);
    // (dS fragment pairs are indexed in 32 bits inside the kernels; the API layer sizes the buffer)
    if (a.dS_frag) {
        if (a.D == 128) bwd_dkdv_kernel_w4<128, true><<<grid, 256, 0, st>>>(k);
        else if (a.D == 80) bwd_dkdv_kernel_w4<80, true><<<grid, 256, 0, st>>>(k);
        else bwd_dkdv_kernel_w4<64, true><<<grid, 256, 0, st>>>(k);
    } else {
        if (a.D == 128) bwd_dkdv_kernel_w4<128, false><<<grid, 256, 0, st>>>(k);
        else if (a.D == 80) bwd_dkdv_kernel_w4<80, false><<<grid, 256, 0, st>>>(k);
        else bwd_dkdv_kernel_w4<64, false><<<grid, 256, 0, st>>>(k);
    }
    if (k.splits == 1) return;
    const dim3 sum_grid(n_wg * 2 * (unsigned)(dpad(a.D) / 32), 2);  // 8 DB accumulator tiles per workgroup, four per block
    if (a.D == 128) dkdv_sum_kernel<128><<<sum_grid, 256, 0, st>>>(k, n_wg);
    else if (a.D == 80) dkdv_sum_kernel<80><<<sum_grid, 256, 0, st>>>(k, n_wg);
    else dkdv_sum_kernel<64><<<sum_grid, 256, 0, st>>>(k, n_wg);
}

// dQ of the launch from the dS fragments that launch_bwd_dkdv wrote for the same ranges
void launch_bwd_dq_from_ds(const BwdArgs& a, hipStream_t st)
{
    const BwdKernelArgs k = to_kernel_args(a);
    const int waves = sweep_waves(a.n_q, a.Hq);  // (the accumulators' layout follows it: the same in every launch of a call)
    const dim3 grid((unsigned)((a.n_q / (32 * waves)) * a.Hq));
#define DQ_DS_LAUNCH(D_)                                                     \
    do {                                                                     \
        if (waves == 8) bwd_dq_ds_kernel<D_, 8><<<grid, 512, 0, st>>>(k);    \
        else if (waves == 4) bwd_dq_ds_kernel<D_, 4><<<grid, 256, 0, st>>>(k); \
        else bwd_dq_ds_kernel<D_, 2><<<grid, 128, 0, st>>>(k);               \
    } while (0)
    if (a.D == 128) DQ_DS_LAUNCH(128);
    else if (a.D == 80) DQ_DS_LAUNCH(80);
    else DQ_DS_LAUNCH(64);
#undef DQ_DS_LAUNCH
}

void launch_bwd_dq(const BwdArgs& a, hipStream_t st)
{
    const BwdKernelArgs k = to_kernel_args(a);
    const int kg = dq_key_groups(a.n_q, a.n_k, a.Hq, a.D, a.q_pos0 == a.k_pos0);
    const dim3 grid((unsigned)((a.n_q / (bwd_q_tile(a.D) / kg)) * a.Hq));
#define DQ_LAUNCH(D_)                                                        \
    do {                                                                     \
        if (kg == 4) bwd_dq_kernel<D_, 4><<<grid, NTHREAD, 0, st>>>(k);      \
        else if (kg == 2) bwd_dq_kernel<D_, 2><<<grid, NTHREAD, 0, st>>>(k); \
        else bwd_dq_kernel<D_, 1><<<grid, NTHREAD, 0, st>>>(k);              \
    } while (0)
    if (a.D == 128) DQ_LAUNCH(128);
    else if (a.D == 80) DQ_LAUNCH(80);
    else DQ_LAUNCH(64);
#undef DQ_LAUNCH
}

void launch_stat_pack(const float* LSE, const float* Delta, int64_t stride, int64_t rows, int Hq,
                      int64_t out_head_stride_blocks, float* out, hipStream_t st)
{
    const int64_t items = rows / 32 * Hq;
    if (items <= 0) return;
    stat_pack_kernel<<<dim3((unsigned)((items + 3) / 4)), 256, 0, st>>>(LSE, Delta, stride, rows / 32, Hq,
                                                                       out_head_stride_blocks, out);
}

void launch_delta(const void* O, const void* dO, int64_t rows, int Hq, int D, int is_bf16,
                  float* Delta, int64_t delta_stride, hipStream_t st, unsigned* clear, int n_clear)
{
    const int64_t pairs = rows * Hq;
    dim3 grid((unsigned)((pairs + 15) / 16));
    if (is_bf16)
        delta_kernel<uint16_t><<<grid, 256, 0, st>>>((const uint16_t*)O, (const uint16_t*)dO, rows, Hq, D, Delta, delta_stride, clear, n_clear);
    else
        delta_kernel<float><<<grid, 256, 0, st>>>((const float*)O, (const float*)dO, rows, Hq, D, Delta, delta_stride, clear, n_clear);
}

void launch_bwd_prepare(const BwdArgs& a, const void* O, float* Delta, float* stat2, void* Qnat, void* dOnat, void* Knat, void* Vnat, hipStream_t st)
{
    PrepareArgs p;
    p.Q = (const uint16_t*)a.Q; p.dO = (const uint16_t*)a.dO; p.K = (const uint16_t*)a.K; p.V = (const uint16_t*)a.V; p.O = (const uint16_t*)O;
    p.LSE = a.LSE; p.Delta = Delta; p.stat2 = stat2;
    p.S = a.n_q; p.Hq = a.Hq; p.Hkv = a.Hkv; p.c = a.scale * LOG2E;
    p.jobs = {{{a.Q, a.Hq, Qnat, nullptr}, {a.dO, a.Hq, dOnat, nullptr}, {a.K, a.Hkv, Knat, nullptr}, {a.V, a.Hkv, Vnat, nullptr}}};
    p.head_blocks = DELTA_HEAD_ROWS / 32 * (unsigned)a.Hq;
    p.delta_blocks = (unsigned)((a.n_q - DELTA_HEAD_ROWS) / 32 * a.Hq);
    const int64_t blocks = bwd_prepare_blocks(a.n_q, a.Hq, a.Hkv);
    for (int64_t first = 0, n; first < blocks; first += n) {
        n = bwd_prepare_next(first, blocks);
        p.first = (unsigned)first;
        if (a.D == 128) bwd_prepare_kernel<128><<<(unsigned)n, 512, 0, st>>>(p);
        else if (a.D == 80) bwd_prepare_kernel<80><<<(unsigned)n, 512, 0, st>>>(p);
        else bwd_prepare_kernel<64><<<(unsigned)n, 512, 0, st>>>(p);
    }
}

void launch_delta_head(const void* Q, const void* dO, const void* K, const void* V, const float* LSE,
                       int64_t stat_stride, int Hq, int Hkv, int D, float scale, float* Delta, hipStream_t st)
{
    const dim3 grid((unsigned)(DELTA_HEAD_ROWS / 32 * Hq));
    const float c = scale * LOG2E;
    const uint16_t *q = (const uint16_t*)Q, *g = (const uint16_t*)dO, *k = (const uint16_t*)K, *v = (const uint16_t*)V;
    if (D == 128) delta_head_kernel<128><<<grid, 512, 0, st>>>(q, g, k, v, LSE, stat_stride, Hq, Hkv, c, Delta);
    else if (D == 80) delta_head_kernel<80><<<grid, 512, 0, st>>>(q, g, k, v, LSE, stat_stride, Hq, Hkv, c, Delta);
    else delta_head_kernel<64><<<grid, 512, 0, st>>>(q, g, k, v, LSE, stat_stride, Hq, Hkv, c, Delta);
}

}  // namespace fpdt
