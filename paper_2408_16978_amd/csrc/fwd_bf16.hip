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
// global -> LDS directly (no register staging).  KG = 1: the waves own 256
// query rows and share the key tiles.  KG = 2, 4: 128 or 64 query rows, the waves of one row block take
// every KG-th 32-key block (or pair of blocks) and merge their (max, sum, output) through LDS at the end, for launches whose
// row tiles are too few to fill the chip or whose longest row tile decides (sweep_key_groups).
//
// us per launch, all waves in one phase at a time and copies behind branches -> this kernel (8 query / 2 KV heads; whole sequences, then
// pairs of chunks): D = 128, 1K 17.2 -> 14.2, 2K 26.2 -> 20.8, 8K 146 -> 137, 64K 7445 -> 7210 (1220 TFLOP/s), 4K chunks 90.5 -> 77.8; D = 80, 2K 20.1 ->
// 17.5, 64K (4 heads) 2774 -> 2639, 8K chunks (4 heads) 126 -> 105; D = 64, 8K 94 -> 84, 64K 4464 -> 4262, 4K chunks 53.8 -> 47.1.
#include <type_traits>

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

// KG key groups: 256 / KG query rows per workgroup of eight waves; the waves of a row block take every KG-th 32-key block and merge
// their (max, sum, output) through LDS at the end.
//
// RAW: K and V come from their row-major tensors instead of packed fragments.  A 32-key block is copied row by row, 16-byte
// piece q of row r at position q ^ swz(r) of its row, swz(r) = 4 (r % 4) + (r / 4) % 4 (D = 64: 4 (r / 2 % 2) + (r / 4) %
// 4; D = 80: rows of ten pieces as they are): the lanes that a fragment read serves at a time, and the four rows of a
// transposing read, lie in different banks.  V's operand is then read with transposing loads, two for one plain
// read.  For short sequences, where the packing launch costs more than these reads (sweep_reads_tensors, launch_rules.h).
//
// A tile is 32 KG keys, and costs a compute unit about the same on its matrix cores, in its LDS, in its vector ALUs and, with four key
// groups, in the unit that addresses the copies; besides, every instruction costs one of the two waves of a SIMD about five clocks.
// So a tile is two phases of straight code, a barrier behind each, whose MFMAs have their operands in registers since the phase
// before and hide everything else, all of it requested or read one at a time between them:
//   A: scores of the NEXT tile's block, exponentials of this one's; reads V of this tile
//   B: O^T += V^T P^T; reads K of tile it + 2
// The two waves of a SIMD (w and w + 4) are one phase apart, so that A's vector work runs under B's MFMAs: in global phases, the early
// waves are in A(it) in 2 it and in B(it) in 2 it + 1, the late ones one later.  LDS holds two tiles of K and two of V; a slot
// is free once both have read it, so V of tile it + 1 is requested in phase 2 it, K of tile it + 3 in 2 it + 1, by all waves, and each
// has landed by the end of the next phase: a wave waits for all but what it requested in the phase that ends.
template <int D, int KG, int KB, int NWAVE, bool RAW>
__global__ __launch_bounds__(NWAVE * 64, 2) void fwd_sweep_kernel(FwdKernelArgs p)
{
    constexpr int DT = D / 16, DP = (D + 31) / 32 * 32, DB = DP / 32;
    constexpr int NB = KG * KB, BK = NB * 32;  // 32-key blocks and keys per LDS tile, KB blocks per group
    constexpr int NQ = NWAVE / KG, BQ = NQ * 32;  // row blocks and query rows per workgroup
    constexpr int VF = RAW ? DT : 2 * DB;   // 1 KiB copies of V per 32-key block
    constexpr int KFRAG = NB * DT, VFRAG = NB * VF;  // copies of K, V per tile
    constexpr bool PAIR = KG == 1 && KB == 1;        // two tiles share a reference and a partial sum, as one of two blocks does
    constexpr int CPP = ((VFRAG > KFRAG ? VFRAG : KFRAG) + NWAVE - 1) / NWAVE;  // copies of a wave per phase
    // (The count of copies is every wave's, so that a phase's wait is one constant: at D = 80 more than there are fragments.  With one key group and
    // eight waves a tile of 22 KiB requests 32, K 16 for 10 fragments, V 16 for 12.  What that costs has not been timed by itself.)
    static_assert(CPP * NWAVE <= 2 * KFRAG && CPP * NWAVE >= VFRAG, "a wave without a fragment of its own copies another's once more");
    constexpr int K_U4 = KFRAG * 64, V_U4 = VFRAG * 64;  // u32x4 per K, V tile
    constexpr int PAD = RAW && DP > D ? 4 : 0;  // the last row's padded channels are read from behind it
    constexpr int SHARE = DB * 16 / KG;         // accumulator registers that a wave of a row block merges in the end
    constexpr int MERGE_U4 = NWAVE * (KG - 1) * (SHARE / 4) * 64;
    constexpr int RING_U4 = 2 * (K_U4 + V_U4) + PAD;
    __shared__ u32x4 ring[RING_U4 > MERGE_U4 ? RING_U4 : MERGE_U4];  // two K tiles, two V tiles; in the end what the waves merge
    __shared__ float ml[KG > 1 ? NWAVE : 1][2][64];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wu = __builtin_amdgcn_readfirstlane(w);
    const int half = lane >> 5, col = lane & 31;
    const int qb = wu % NQ, kg = wu / NQ;  // this wave's row block and its share of the key blocks
    const int head = blockIdx.x % p.Hq;
    const int n_qt = p.n_q / BQ;
    const int qt = n_qt - 1 - (int)(blockIdx.x / p.Hq);  // heaviest (latest) tiles first
    const int kvh = head / p.g;
    const int q0 = qt * BQ;       // first row of the workgroup within the launch
    const int qw0 = q0 + qb * 32;  // first row of this wave

    // keys this workgroup needs: positions <= last query position
    const int ahead_pos = (int)(p.q_pos0 - p.k_pos0) + q0;  // position of the workgroup's first row behind the launch's first key (below 2^30)
    const int need = ahead_pos + BQ < p.n_keys ? ahead_pos + BQ : p.n_keys;
    const int n_tiles = (need + BK - 1) / BK;

    // This lane's reads of the wave's block of a tile: K's fragments, V's transposing loads (RAW) or V's fragments, as LDS addresses within
    // slot 0, and its bytes of the wave's copies, from the tile's first byte on.  All of them are in registers: an instruction costs
    // a wave of these workgroups, two of which share a SIMD, about five clocks, whatever it does.
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef short short8v __attribute__((ext_vector_type(8)));
    typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;
    typedef __attribute__((address_space(3))) u32x4* lds_u32x4_ptr;
    typedef __attribute__((address_space(3))) char* lds_byte_ptr;
    constexpr int PPR = D / 8, ROW = 2 * D;  // pieces and bytes of a row
    const unsigned ring_lds = lds_address(ring);
    auto swz = [](int r) { return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : D == 64 ? (((r >> 1) & 1) << 2) | ((r >> 2) & 3) : 0; };
    constexpr int K_READS = RAW && D != 80 ? DT : 1, V_READS = !RAW ? 1 : D == 80 ? 2 : 2 * DB;
    unsigned k_at[K_READS], v_at[V_READS];
    {
        const unsigned kb = ring_lds + 1024u * (unsigned)(kg * KB * DT), vb = ring_lds + 32u * K_U4 + 1024u * (unsigned)(kg * KB * VF);
#pragma unroll
        for (int t = 0; t < K_READS; ++t) k_at[t] = kb + (RAW ? (unsigned)(col * ROW + 16 * (half ^ swz(col))) ^ (32u * (unsigned)t) : 16u * (unsigned)lane);
        const int grp = lane >> 4, h = grp >> 1, dblk = grp & 1, e = (lane & 15) >> 2, x = lane & 3;
#pragma unroll
        for (int i = 0; i < V_READS; ++i) {  // load I = i % 2 of channel block i / 2
            const int r = 8 * (i % 2) + 4 * h + e;
            const unsigned at = (unsigned)(r * ROW + 16 * ((2 * dblk + (x >> 1)) ^ swz(r)) + 8 * (x & 1));
            v_at[i] = vb + (RAW ? at ^ (64u * (unsigned)(i / 2)) : 16u * (unsigned)lane);
        }
    }
    // (opaque: the compiler would rather add them up again than keep them)
#pragma unroll
    for (int t = 0; t < K_READS; ++t) asm("" : "+v"(k_at[t]));
#pragma unroll
    for (int i = 0; i < V_READS; ++i) asm("" : "+v"(v_at[i]));
    // Copies: those of phase A (of V for early waves, of K for late ones) and of phase B (the other).  Copy i of a wave is fragment
    // w + NWAVE i of the tile.
    const bool late = NWAVE == 8 && wu >= 4;
    const unsigned pitch = RAW ? (unsigned)p.kv_pitch * 2u : 0u;
    struct Copies {
        uint64_t src, step;   // of the tile that is requested next; from tile to tile
        unsigned dst, other;  // LDS slots: of that tile, of the one after it
        unsigned at[CPP], lane_off[CPP];
    } cp[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const bool of_k = (k == 0) == late;
        const int n = of_k ? KFRAG : VFRAG;
#pragma unroll
        for (int i = 0; i < CPP; ++i) {
            const int f = NWAVE * i + wu < n ? NWAVE * i + wu : NWAVE * i + wu - n;
            cp[k].at[i] = 1024u * (unsigned)f;
            if constexpr (RAW) {
                const int blk = f / DT, piece = 64 * (f - blk * DT) + lane, r = D == 80 ? (piece * 6554) >> 16 : piece / PPR;
                cp[k].lane_off[i] = (unsigned)(32 * blk + r) * pitch + 16u * (unsigned)((piece - r * PPR) ^ swz(r));
            } else {
                cp[k].lane_off[i] = 1024u * (unsigned)f + 16u * (unsigned)lane;
            }
        }
        if constexpr (RAW) {
            cp[k].src = uniform((uint64_t)(uintptr_t)(of_k ? p.K : p.V) + (uint64_t)kvh * ROW);
            cp[k].step = (uint64_t)BK * pitch;
        } else {
            cp[k].src = uniform((uint64_t)(uintptr_t)(of_k ? p.Knat : p.Vtr) + (uint64_t)kvh * p.kv_head_stride_blocks * (of_k ? DT * 1024 : 2 * DB * 1024));
            cp[k].step = of_k ? K_U4 * 16 : V_U4 * 16;
        }
        cp[k].dst = ring_lds + (of_k ? 0u : 32u * K_U4);
        cp[k].other = cp[k].dst + 16u * (of_k ? K_U4 : V_U4);
    }
    auto next = [](Copies& c) {
        c.src += c.step;
        const unsigned d = c.dst;
        c.dst = c.other;
        c.other = d;
    };
    auto request = [&](Copies& c) {
#pragma unroll
        for (int i = 0; i < CPP; ++i) copy_1k(c.src, c.dst, c.at[i], c.lane_off[i]);
        next(c);
    };
    const int a_ahead = late ? 3 : 1, b_ahead = late ? 2 : 3;  // the tile that phase A, B of tile `it` requests: it + ..

    // Q fragments (B operand of S^T = K Q^T): lane (col, half) holds Q[row][16t + 8 half + e]
    bf16x8 qf[DT];
    {
        const uint16_t* qrow = p.Q + ((size_t)(qw0 + col) * p.Hq + head) * D + 8 * half;
#pragma unroll
        for (int t = 0; t < DT; ++t) qf[t] = as_bf16x8(*reinterpret_cast<const u32x4*>(qrow + 16 * t));
    }

    floatx16 acc[DB];
    float m_run, l_run;  // l_run is this lane's partial sum (its 16 keys per block)
    float pair_sum = 0.f;  // PAIR: of the even tile, until the odd one's joins it
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

    if (late) {
        request(cp[0]);
        request(cp[1]);
        if (n_tiles > 1) request(cp[0]);
    } else {
        request(cp[1]);
        request(cp[0]);
        if (n_tiles > 1) request(cp[1]);
    }
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

    const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // tiles in which this wave has a key at or below its diagonal: the first n_w
    const int reach = ahead_pos + 32 * (qb - kg * KB);  // of the wave's first row behind its first key
    const int n_w = reach + 31 < 0 ? 0 : (reach + 31) / BK + 1 < n_tiles ? (reach + 31) / BK + 1 : n_tiles;
    const int row_key = reach + col - 4 * half;  // the last key this lane's query sees, from the wave's first key on, less the lane's offset

    // fragments of the wave's block of the tile in a slot
    auto read_k = [&](auto from, int kb, int t) -> bf16x8 {
        const unsigned SLOT = decltype(from)::value * K_U4 * 16 + 1024u * (unsigned)(kb * DT);
        return as_bf16x8(*(lds_u32x4_ptr)((lds_byte_ptr)(uintptr_t)k_at[K_READS > 1 ? t : 0] + (SLOT + (K_READS > 1 ? 0u : (RAW ? 32u : 1024u) * (unsigned)t))));
    };
    auto read_v = [&](auto from, int kb, int s2, int db) -> bf16x8 {
        const unsigned SLOT = decltype(from)::value * V_U4 * 16 + 1024u * (unsigned)(kb * VF);
        if constexpr (RAW) {
            const unsigned at = SLOT + (unsigned)(16 * s2 * ROW);
            auto part = [&](int I) {
                return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)((lds_byte_ptr)(uintptr_t)v_at[D == 80 ? I : 2 * db + I] + (at + (D == 80 ? 64u * (unsigned)db : 0u))));
            };
            const short8v both = __builtin_shufflevector(part(0), part(1), 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        } else {
            return as_bf16x8(*(lds_u32x4_ptr)((lds_byte_ptr)(uintptr_t)v_at[0] + (SLOT + 1024u * (unsigned)(s2 * DB + db))));
        }
    };
    // end of a phase: all copies of this wave but those that the phase has requested have landed
    auto end_phase = [&](bool requested) {
        if (requested) wait_vmem_at_most<CPP>();
        else wait_vmem_at_most<0>();
        barrier_no_fence();
    };

    constexpr std::integral_constant<int, 0> ZERO{};
    constexpr std::integral_constant<int, 1> ONE{};

    // before the first tile: its scores, K of the second in registers
    floatx16 s[KB];
    bf16x8 kfr[KB][DT];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
        for (int t = 0; t < DT; ++t) kfr[kb][t] = read_k(ZERO, kb, t);
#pragma unroll
        for (int t = 0; t < DT; ++t) s[kb] = mfma32(kfr[kb][t], qf[t], t == 0 ? zero : s[kb]);
    }
#pragma unroll
    for (int i = 0; i < KB * DT; ++i) kfr[i % KB][i / KB] = read_k(ONE, i % KB, i / KB);
    barrier_no_fence();
    if (n_tiles > 2) {
        if (late) request(cp[0]);
        else request(cp[1]);
    }
    if (late) {
        if (n_tiles > 1) request(cp[1]);
        end_phase(n_tiles > 1);
    }

    // Tile `it`, of parity `par`: V in slot par, K of tile it + 2 too.  STEADY: both phases have something to request, and copies go out between
    // the MFMAs of straight code.  (With a branch around each copy the compiler moves the exponentials behind the last of them.)
    auto tile = [&](auto steady, int it, auto par) {
        constexpr bool STEADY = decltype(steady)::value;
        const bool more_a = STEADY || it + a_ahead < n_tiles, more_b = STEADY || it + b_ahead < n_tiles;
        if (it * BK + 32 * KB - 1 > reach) {  // wave-uniform: the tile straddles the diagonal
            const int last = row_key - it * BK;  // a key is masked when 32 kb + 8 (r / 4) + r % 4 + 4 half > query - first key
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (32 * kb + 8 * (r >> 2) + (r & 3) > last) s[kb][r] = -INFINITY;
        }
        // ---- A.  (Behind the wave's last block the scores are of whatever the registers hold, and never used.) ----
        // The running maximum is only a reference point: any value gives the same O and LSE as
        // long as nothing overflows.  So the block is exponentiated against the reference it
        // found, optimistically, and no maximum is taken at all; the row sums that are needed
        // anyway tell when that was wrong: every probability is at most the partial sum it
        // went into, so a sum within REF_LIMIT (far inside the range of bf16 and of the fp32
        // sums) proves that no probability exceeded it.  A sum beyond it -- or infinite, or not
        // a number, as on a row's first block, where the reference is still -inf -- sends the
        // whole wave through the exact path below (true maximum, rescale, exponentiate again):
        // a row's first block, and later only when its maximum rises by more than 14 in log2.
        constexpr float REF_LIMIT = 16384.f;
        constexpr int VR = KB * 2 * DB, AS = KB * DT;  // V fragments of the tile = MFMAs of phase B; MFMAs of phase A
        bf16x8 vfr[VR], pf[KB][2];
        floatx16 ahead[KB];
        constexpr bool FIRST = PAIR && decltype(par)::value == 0, SECOND = PAIR && decltype(par)::value == 1;
        float lsum = SECOND ? pair_sum : 0.f;
        {
            if (!STEADY && more_a) request(cp[0]);
            floatx16 e[KB];
            for_each<AS>([&](auto step) {
                constexpr int j = decltype(step)::value, t = j / KB, kb = j % KB;
                ahead[kb] = mfma32(kfr[kb][t], qf[t], t == 0 ? zero : ahead[kb]);
#pragma unroll
                for (int i = reads_before(j, AS, VR); i < reads_before(j + 1, AS, VR); ++i) vfr[i] = read_v(par, i / (2 * DB), i / DB % 2, i % DB);
#pragma unroll
                for (int i = CPP * j / AS; STEADY && i < CPP * (j + 1) / AS; ++i) copy_1k(cp[0].src, cp[0].dst, cp[0].at[i], cp[0].lane_off[i]);
#pragma unroll
                for (int r = 16 * KB * j / AS; r < 16 * KB * (j + 1) / AS; ++r) {
                    e[r / 16][r % 16] = __builtin_amdgcn_exp2f(fmaf(s[r / 16][r % 16], p.c, -m_run));
                    lsum += e[r / 16][r % 16];
                    if (r % 16 == 7) pf[r / 16][0] = pack_half<0>(e[r / 16]);
                    if (r % 16 == 15) pf[r / 16][1] = pack_half<1>(e[r / 16]);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            if (STEADY) next(cp[0]);
        }
        if (__any(!(lsum <= REF_LIMIT))) {
            float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
            for (int r = 2; r < 16 * KB; r += 2) mx = fmaxf(fmaxf(mx, s[r / 16][r % 16]), s[r / 16][r % 16 + 1]);
            if constexpr (FIRST) {
                // The next block's scores are here too, and count: the largest probability of a reference is exact in bf16, and of the
                // first 64 keys, which make up the short rows, it is so in more rows than of the first 32 (8 heads, 16K tokens: error of
                // O against 64 bits 2.168e-3 with 32, 2.154e-3 with 64; sums of 64 keys: of the LSE 5.4e-8, 5.3e-8).
                int last = row_key - (it + 1) * BK;
                asm volatile("" : "+v"(last));  // (the comparisons stay in the branch)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + (r & 3) <= last) mx = fmaxf(mx, ahead[0][r]);
            }
            mx = fmaxf(mx, xor32(mx));
            const float mc = mx * p.c;
            const float m_new = mc > m_run ? mc : m_run;  // (a lane whose keys are all masked keeps its reference)
            // (a row may have had no key in this wave's blocks yet; its reference stays at -inf, and 0 takes its place in
            // the exponents)
            const float m_exp = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_exp);  // 0 on a row's first block, 1 where nothing moved
            if (SECOND) l_run += pair_sum;
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
        if (!FIRST) l_run += lsum;
        if (PAIR) pair_sum = FIRST ? lsum : 0.f;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) s[kb] = ahead[kb];
        end_phase(more_a);
        // Where the second block lies behind all of the wave's rows (only ever in its last tile, which is no steady one) its probabilities are 0:
        // its V counts as 0 too, so that an infinity or NaN there does not reach rows of the block before.
        if constexpr (KB == 2 && !STEADY)
            if (it * BK + 32 > reach + 31) {  // wave-uniform
#pragma unroll
                for (int i = 2 * DB; i < VR; ++i) vfr[i] = as_bf16x8(u32x4{0, 0, 0, 0});
            }
        // ---- B ----
        if (!STEADY && more_b) request(cp[1]);
        for_each<VR>([&](auto step) {
            constexpr int j = decltype(step)::value;
            acc[j % DB] = mfma32(vfr[j], pf[j / (2 * DB)][j / DB % 2], acc[j % DB]);
#pragma unroll
            for (int i = reads_before(j, VR, AS); i < reads_before(j + 1, VR, AS); ++i) kfr[i % KB][i / KB] = read_k(par, i % KB, i / KB);
#pragma unroll
            for (int i = CPP * j / VR; STEADY && i < CPP * (j + 1) / VR; ++i) copy_1k(cp[1].src, cp[1].dst, cp[1].at[i], cp[1].lane_off[i]);
            __builtin_amdgcn_sched_barrier(0);
        });
        if (STEADY) next(cp[1]);
        end_phase(more_b);
    };
    int it = 0;
#pragma unroll 1
    for (; it + KB < n_w && it + 4 < n_tiles; it += 2) {
        tile(std::true_type{}, it, ZERO);
        tile(std::true_type{}, it + 1, ONE);
    }
#pragma unroll 1
    while (it < n_w) {
        tile(std::false_type{}, it++, ZERO);
        if (it < n_w) tile(std::false_type{}, it++, ONE);
    }
#pragma unroll 1
    for (; it < n_tiles; ++it) {  // tiles of later rows of the workgroup: this wave's share of the copies
        if (it + a_ahead < n_tiles) request(cp[0]);
        end_phase(it + a_ahead < n_tiles);
        if (it + b_ahead < n_tiles) request(cp[1]);
        end_phase(it + b_ahead < n_tiles);
    }
    if (NWAVE == 8 && !late) barrier_no_fence();  // the late waves' last phase
    l_run += pair_sum;

    if (p.flags & SWEEP_FINAL) {
        // Merge the waves of a row block: each its share of the registers, so that all of them read and store.  (Every copy has
        // landed and every wave is past the last barrier: nobody reads the ring any more.)
        if (KG > 1) {
            ml[wu][0][lane] = m_run;
            ml[wu][1][lane] = l_run;
        }
        floatx4* const part = reinterpret_cast<floatx4*>(ring) + lane;
        auto at = [&](int owner, int from, int i) {  // `from`: which of the owner's KG - 1 others
            return (size_t)(((qb * KG + owner) * (KG - 1) + from) * (SHARE / 4) + i) * 64;
        };
        auto quad = [&](int j) {  // accumulator registers 4 j .. 4 j + 3: channels 8 j + 4 half + 0..3
            floatx4 v;
#pragma unroll
            for (int b = 0; b < 4; ++b) v[b] = acc[j / 4][4 * (j % 4) + b];
            return v;
        };
#pragma unroll
        for (int owner = 0; owner < KG; ++owner)
            if (owner != kg) {
#pragma unroll
                for (int i = 0; i < SHARE / 4; ++i) part[at(owner, kg - (kg > owner), i)] = quad(owner * (SHARE / 4) + i);
            }
        if (KG > 1) __syncthreads();
        float m_all = -INFINITY, l_all = 0.f, wt[KG];
#pragma unroll
        for (int i = 0; i < KG; ++i) m_all = fmaxf(m_all, KG > 1 ? ml[i * NQ + qb][0][lane] : m_run);
#pragma unroll
        for (int i = 0; i < KG; ++i) {
            // (0 in the place of a maximum of -infinity: a row that scores nothing else has a sum of 0 then, with every key group count)
            wt[i] = KG > 1 ? __builtin_amdgcn_exp2f(ml[i * NQ + qb][0][lane] - (m_all > -INFINITY ? m_all : 0.f)) : 1.f;
            l_all += KG > 1 ? ml[i * NQ + qb][1][lane] * wt[i] : l_run;
        }
        const float l_tot = l_all + xor32(l_all), inv = 1.f / l_tot;
        const int row = qw0 + col;
        uint16_t* orow = p.O + ((size_t)row * p.Hq + head) * D;
#pragma unroll
        for (int owner = 0; owner < KG; ++owner)
            if (owner == kg) {
#pragma unroll
                for (int i = 0; i < SHARE / 4; ++i) {
                    const int j = owner * (SHARE / 4) + i, d = 8 * j + 4 * half;
                    floatx4 v = quad(j) * wt[owner];
#pragma unroll
                    for (int from = 0; from < KG - 1; ++from) v += part[at(owner, from, i)] * wt[from + (from >= owner)];
                    v *= inv;
                    if (8 * j < D) *reinterpret_cast<bf16x4*>(orow + d) = __builtin_convertvector(v, bf16x4);
                }
            }
        if (half == 0 && kg == 0) p.LSE[(size_t)head * p.lse_stride + row] = (m_all + __builtin_log2f(l_tot)) * LN2;
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
        constexpr int KB_ = D_ == 128 ? 1 : 2;                                                      \
        const dim3 grid((unsigned)((a.n_q / (waves * 32 / kg)) * a.Hq));                            \
        if (kg == 4 && a.K) fwd_sweep_kernel<D_, 4, 1, 8, true><<<grid, 512, 0, st>>>(k);           \
        else if (kg == 4) fwd_sweep_kernel<D_, 4, 1, 8, false><<<grid, 512, 0, st>>>(k);            \
        else if (kg == 2 && a.K) fwd_sweep_kernel<D_, 2, KB_, 8, true><<<grid, 512, 0, st>>>(k);    \
        else if (kg == 2) fwd_sweep_kernel<D_, 2, KB_, 8, false><<<grid, 512, 0, st>>>(k);          \
        else if (waves == 8) fwd_sweep_kernel<D_, 1, KB_, 8, false><<<grid, 512, 0, st>>>(k);       \
        else fwd_sweep_kernel<D_, 1, KB_, 4, false><<<grid, 256, 0, st>>>(k);                       \
    } while (0)
    if (a.D == 128) FWD_LAUNCH(128);
    else if (a.D == 80) FWD_LAUNCH(80);
    else FWD_LAUNCH(64);
#undef FWD_LAUNCH
}

}  // namespace fpdt
