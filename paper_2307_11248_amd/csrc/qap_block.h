// qap_block.h -- block form of the tabu and 2opt searches: one workgroup per search, the
// neighbourhood held as 32 x 32 blocks in matrix-core accumulators, the two long parts of
// an iteration run side by side on different waves.
//
// Why.  With a lane per register tile and a lane per row recomputation (qap_search.hip) the
// same waves did, one after the other, the select, the recomputation of the rows of the
// exchanged pair and the update of the tiles: an iteration was one chain of about 570
// instructions (a wave issues one about every 8 clocks), and two thirds of the vector
// instructions of a tile were the update and the tabu tests of its slots.  Here
//   * the update Delta += (A_u - A_v)(B_u - B_v) + (C_u - C_v)(E_u - E_v) of a 32 x 32
//     block is one v_mfma_i32_32x32x32_i8 into the accumulators that hold the block: a
//     form of rank 6 in 8-bit limbs, 20 of the 32 terms used (W below);
//   * the recomputed deltas of rows r and s are a contraction too: a task wave takes 32 or 64
//     indices u and gets Delta(u, r), Delta(u, s) from v_mfma_i32_16x16x64_i8 on the rows of G
//     and D against the rows r and s, and on their columns (through transposing LDS reads, so
//     no transposed copy is kept) against columns r and s, with one correction product each;
//   * the tabu state of a slot is an offset in its value, so the select of a block is a
//     signed minimum (the free slots) and an unsigned minimum (the tabu ones) of the
//     same keys, with no test per slot.
//
// Waves.  NB = ceil(n / 32).  Task waves (half a wave each for the sides r and s), one
// housekeeping wave, and the block waves, BPW blocks (I <= J) each (Shape).
//
// Matrices are int8, entries minus 128 (zero past n): every delta of Eq. (2) is unchanged
// when a constant is added to all entries of F or of D, so nothing is corrected for it
// except the cost itself, once.
//
// With G = F[p][p], T = G.D^T + G^T.D and SD_u = T_uu, the delta of Eq. (2) is
//   delta(i, j) = T_ij + T_ji - SD_i - SD_j + (d_ij + d_ji - d_ii - d_jj)(g_ij + g_ji - g_ii - g_jj)
// (the six products of the k = i, j terms factor into one).
//
// One iteration, made at `it` (r, s the exchanged pair, p' the permutation after it):
//   B1      the minimum over the waves is in sel[it & 1] (LDS, 64-bit atomic minimum)
//   A       task waves  bytes of rows and columns r and s of D and G for their u; W_u; G
//                       follows the move (rows and columns r, s exchanged in place)
//           block waves the rows and columns of the move before this one take the deltas
//                       the task waves recomputed then; tabu moves that expire are freed
//           housekeeping the corner entries of G; tabu bits and ring; best-so-far
//   B2
//   B       task waves  Delta'(u, r), Delta'(u, s) under p', their candidate for it + 1
//           block waves one MFMA a block, candidate of every slot outside r and s
//           housekeeping p; the tabu moves that expire at it + 2
// The rows and columns of r and s in the blocks are stale between B and the next A and are
// left out of the blocks' minimum; the task waves' candidates stand for them.
//
// Bound by the chain of an iteration (two barriers, about 0.9 us up to n = 96), from n = 160 on by
// the task waves' waits for LDS.  At n = 256 their reads (2 n^2 bytes for each of rows and
// columns, 128 a clock) and products are 0.85 and 0.5 us of 3.5: a wave of two groups (TC = 2)
// asks for the operands of a half step, waits and multiplies, eight times, with nothing of the
// next half step on its way (waves wait 0.55 of their cycles and issue in 0.25).  us per
// iteration, tiles (qap_search.hip) and here, one search a compute unit: n = 40 2.0 and 1.0,
// n = 64 1.9 and 0.9, n = 128 symmetric 2.4 and 1.2, n = 256 17.7 and 3.5; 4096 searches of
// uneven n up to 150: 29.6 and 16.7 ms for 1000 iterations.
#pragma once

#include "qap_internal.h"

namespace qapk {

namespace {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef short short2_t __attribute__((ext_vector_type(2)));

// A slot holds delta - BK_OFF while its move may be made and delta + BK_OFF while it is
// tabu (|delta| <= (2n - 2) 255 * 127 < 2^24 for the instances served here): 27 bits, so
// slot * 32 + (row in the block) is a 32-bit key whose sign says whether it is tabu.
constexpr int BK_OFF = 1 << 25;
constexpr int BK_NOMOVE = (1 << 26) - 1;   // diagonal and padding: above every key, both ways
constexpr long long BK_NONE = ((long long)INT32_MAX << 32) | (unsigned)KEY_NONE;

template <int NB>
struct Shape {
    // blocks per block wave (consecutive in (I, J) order) and 32-index groups per task wave:
    // the fewest of both that keep the workgroup within 16 waves
    static constexpr int NBLK = NB * (NB + 1) / 2;
    static constexpr int BPW = NB <= 4 ? 1 : (NB == 5 ? 2 : (NB <= 7 ? 3 : 4));
    static constexpr int TC = NB <= 6 ? 1 : 2;
    static constexpr int TW = (NB + TC - 1) / TC;     // task waves
    static constexpr int BW = (NBLK + BPW - 1) / BPW; // block waves
    static constexpr int WAVES = TW + 1 + BW;
    static_assert(WAVES <= 16, "one workgroup");
    static constexpr int LANES = WAVES * 64;
    static constexpr int KS = (NB + 1) / 2;           // 64-byte steps of a row
    // n above 224: rows of exactly 256 bytes, their 16-byte columns exchanged by the row
    // (column ^ row % 16), since a padded row would not leave LDS for the rest
    static constexpr bool SW = NB == 8;
};

// LDS row stride: an odd multiple of 16 bytes, so 16 consecutive rows start in 16 different
// 16-byte columns of the banks.
__host__ __device__ inline int blk_stride(int n) { return n > 224 ? 256 : (((n + 15) / 16) | 1) * 16; }

// Rows staged: whole 16-row steps, zero past n.
__host__ __device__ inline int blk_rows(int n) { return (n + 15) & ~15; }

struct BlkPlan {
    int g, d, w, rp, perm, bestp, bits, ring, side, total;
};

__host__ __device__ inline int blk_ring(int hi) {
    int r = 32;
    while (r < hi + 2) r *= 2;
    return r;
}

__host__ __device__ inline BlkPlan blk_plan(int n, int nb, int sym, int hi, bool tabu) {
    const int rs = blk_stride(n), np = nb * 32;
    BlkPlan q;
    int o = 0;
    auto take = [&o](int bytes) { int at = o; o += (bytes + 15) & ~15; return at; };
    q.g = take(blk_rows(n) * rs);
    q.d = take(blk_rows(n) * rs);
    q.w = take(np * 32);      // also what a row's last 64-byte step may read past the matrices
    q.rp = take(np * 2 * 4);
    q.perm = take(np * 4);
    q.bestp = take(np * 4);
    q.bits = take(tabu ? np * nb * 4 : 0);
    q.ring = take(tabu ? blk_ring(hi) * 4 : 0);
    q.side = take(sym ? 0 : 4 * 64 * ((nb + 1) / 2));   // columns r, s of D, then of G
    q.total = o;
    return q;
}

__device__ inline int bperm(unsigned hi, unsigned lo, unsigned sel) { return (int)__builtin_amdgcn_perm(hi, lo, sel); }

__device__ inline int pk_sub(int a, int b) {
    return __builtin_bit_cast(int, (short2_t)(__builtin_bit_cast(short2_t, a) - __builtin_bit_cast(short2_t, b)));
}
__device__ inline int pk_add(int a, int b) {
    return __builtin_bit_cast(int, (short2_t)(__builtin_bit_cast(short2_t, a) + __builtin_bit_cast(short2_t, b)));
}
template <int S>
__device__ inline int pk_ashr(int a) {
    return __builtin_bit_cast(int, (short2_t)(__builtin_bit_cast(short2_t, a) >> (short)S));
}
__device__ inline int dot2(int a, int b, int c) {
    return __builtin_amdgcn_sdot2(__builtin_bit_cast(short2_t, a), __builtin_bit_cast(short2_t, b), c, false);
}
__device__ inline int pack16(int lo, int hi) { return bperm((unsigned)hi, (unsigned)lo, 0x05040100u); }

// Minimum of a signed 32-bit value over the wave: DPP row shifts and row broadcasts; lanes
// that shift in from outside a row see INT32_MAX.
__device__ inline int wmin32(int v) {
    constexpr int I = INT32_MAX;
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x111, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x112, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x114, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x118, 0xF, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x142, 0xA, 0xF, false));
    v = min(v, __builtin_amdgcn_update_dpp(I, v, 0x143, 0xC, 0xF, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// Tenures, 64 at a time (one a lane): uniform in [lo, hi] from the first word of
// Philox4x64-10 (Salmon et al., SC'11), key (seed, 0), counter (iteration, start, 0, 0).  The
// ten rounds can be made one by one, a few instructions of each of ten iterations.
struct Tenures {
    unsigned long long c0, c1, c2, c3, k0, k1;
    __device__ void begin(unsigned long long seed, long long it, long long start) {
        c0 = (unsigned long long)it;
        c1 = (unsigned long long)start;
        c2 = c3 = k1 = 0;
        k0 = seed;
    }
    __device__ void round() {
        const unsigned long long M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
        const unsigned long long hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        const unsigned long long hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
        k0 += 0x9E3779B97F4A7C15ULL;
        k1 += 0xBB67AE8584CAA73BULL;
    }
    __device__ int value(int lo, int hi) const {
        const unsigned long long span = (unsigned long long)((long long)hi - lo + 1);
        return lo + (int)(((c0 >> 32) * span) >> 32);
    }
};

// In a uniform branch that is seldom taken: keeps the compiler from computing both sides of
// it and selecting (the sixteen slots of a block each time).
__device__ inline void stay_branch() { asm volatile(""); }

// A barrier behind the wave's own LDS operations (lgkmcnt 0).  __syncthreads alone asks for that
// wait in a form that the compiler may take out where nothing is in flight, and it takes it out of
// the head of a loop whose entry has nothing in flight though the loop's own end has: waves then
// passed B1 with the minimum, the recomputed deltas or the expiring moves of others still on their
// way to LDS.  This one stays.
__device__ inline void block_sync() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __syncthreads();
}

// waits for the wave's own global stores and atomics (vmcnt 0)
__device__ inline void vm_done() { __builtin_amdgcn_s_waitcnt(0x0f70); }

// (called by one lane; the address is opaque, so that no cross-lane reduction is put around it)
__device__ inline void sel_min(long long *slot, int d, int key) {
    int z = 0;
    asm volatile("" : "+v"(z));
    slot += z;
    __hip_atomic_fetch_min(slot, ((long long)d << 32) | (unsigned)key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The small LDS variables of a search (of the kernel, so that one with several forms holds
// them once).
struct BlkShared {
    long long sel[2];      // the minimum over the waves, by iteration parity
    long long red[8];
    int ev[68];            // the number of pairs that become free, then the pairs
    int bad, chunk_end;
};

// FREQ: tabu that keeps the frequency memory (a.freq), for a.attr 1 with marked units in place
// of tabu pairs.
template <int NB, bool SYM, bool TABU, bool RESUME, bool BUSY, bool FREQ>
__device__ __attribute__((always_inline)) void block_body(const Item &a, unsigned char *sm, BlkShared &sh) {
    static_assert((TABU || !RESUME) && (!FREQ || (TABU && !RESUME && !BUSY)), "forms in use");
    using SH = Shape<NB>;
    constexpr int KS = SH::KS, L = SH::LANES, TW = SH::TW, TC = SH::TC, BPW = SH::BPW, NP = NB * 32;
    constexpr bool SW = SH::SW;
    static_assert(TW <= 8, "sh.red");
    long long *const sel = sh.sel, *const s_red = sh.red;
    int *const s_ev = sh.ev;
    int &s_bad = sh.bad, &s_chunk_end = sh.chunk_end;
    const int n = a.n, rs = blk_stride(n), grs = row_stride(n), t = threadIdx.x, lane = t & 63;
    const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
    if (RESUME && wid >= SH::WAVES) return;         // (one workgroup size for every NB there)
    const int half = lane >> 5, l5 = lane & 31;
    const int hi = TABU ? a.hi : 0, lo = TABU ? a.lo : 0;
    const BlkPlan P = blk_plan(n, NB, SYM, hi, TABU);
    const int rmask = blk_ring(hi) - 1;
    int8_t *const smb = reinterpret_cast<int8_t *>(sm);
    int8_t *const G = smb + P.g, *const D = smb + P.d;
    int8_t *const side = smb + P.side;   // (!SYM) D's columns r and s, then G's under p', 64 KS bytes each
    v4i *const Wv = reinterpret_cast<v4i *>(sm + P.w);   // two 16-byte halves per index
    int *const rp = reinterpret_cast<int *>(sm + P.rp);
    int *const perm = reinterpret_cast<int *>(sm + P.perm), *const bestp = reinterpret_cast<int *>(sm + P.bestp);
    unsigned *const bits = reinterpret_cast<unsigned *>(sm + P.bits);
    int *const ring = reinterpret_cast<int *>(sm + P.ring);
    // unit marking: until when the unit at a location is marked (the pairs' bits are not used
    // then); a slot is tabu while either of its units is
    const bool marks = FREQ && a.attr == 1;
    int *const mark = reinterpret_cast<int *>(sm + P.bits);
    SearchState *const st = RESUME ? a.st : nullptr;
    const bool resume = RESUME && st->it > 1;

    // LDS matrices: byte (row, col) is at row * rs + (col ^ sx(row))
    auto sx = [](int row) -> int { return SW ? (row & 15) << 4 : 0; };
    auto at = [&](int row, int col) -> int { return row * rs + (col ^ sx(row)); };
    // 16 bytes of row operands: base from at(row, 16-byte column below 64), then 64-byte steps
    auto step = [](int base, int ks) -> int { return SW ? base ^ (64 * ks) : base + 64 * ks; };
    auto lds16 = [](const int8_t *m, int o) -> v4i { return *reinterpret_cast<const v4i *>(m + o); };
    // 16 rows (from row 16-byte step `k`) of column `col` (a multiple of 16, plus the lane's
    // l % 16): two transposing reads of 8 rows; a lane addresses half a row of 16 columns
    const int trow = (lane & 15) >> 1, tcol = (lane & 1) * 8;
    auto cols16 = [&](const int8_t *m, int k, int col) -> v4i {
        typedef __attribute__((address_space(3))) v2i *lds2;
        const v2i x = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds2)(m + at(k + trow, col + tcol)));
        const v2i y = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds2)(m + at(k + trow + 8, col + tcol)));
        return v4i{x[0], x[1], y[0], y[1]};
    };

    // ---- read and check the start
    if (t == 0) s_bad = s_chunk_end = 0;
    for (int u = t; u < NP; u += L) rp[u] = -1;
    for (int i = t; i < NP * 8; i += L) reinterpret_cast<int *>(Wv)[i] = 0;
    if (TABU) {
        for (int i = t; i < NP * NB; i += L) bits[i] = 0;
        for (int i = t; i <= rmask; i += L) ring[i] = resume ? a.st_ring[i] : -1;
    }
    if (!SYM)
        for (int i = t; i < 4 * 64 * KS / 4; i += L) reinterpret_cast<int *>(side)[i] = 0;
    if (t < 2) sel[t] = BK_NONE;
    if (FREQ) {
        if (t == 0) s_ev[0] = 0;
        for (int i = t; i < a.m; i += L) a.freq[i] = 0;
        vm_done();   // before the adds of the housekeeping wave
    }
    block_sync();
    const int32_t *const pin = resume ? a.st_perm : a.perm_in;
    for (int u = t; u < n; u += L) {
        const int v = pin[u];
        perm[u] = v;
        bestp[u] = resume ? a.st_bestp[u] : v;
        if (v < 0 || v >= n || atomicExch(&rp[v], u) != -1) s_bad = 1;
    }
    block_sync();
    if (s_bad) {
        if (a.perm_out != a.perm_in)
            for (int u = t; u < n; u += L) a.perm_out[u] = pin[u];
        if (t == 0) {
            *a.cost_out = INT64_MIN;
            if (a.steps_out) *a.steps_out = -2;  // QAP_E_NOT_PERM
            if (RESUME) st->done = 1;
        }
        return;
    }

    // ---- stage D and gather G = F[p][p] (entries minus 128, zero past n)
    {
        const uint8_t *const mats = a.mats;
        const int vpr = rs / 16, nr = blk_rows(n);
        for (int i = t; i < nr * vpr; i += L) {
            const int row = i / vpr, c = (i - row * vpr) * 16;
            unsigned m[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int real = n - (c + 4 * e);
                m[e] = real >= 4 ? 0x80808080u : (real <= 0 ? 0u : (0x80808080u >> (8 * (4 - real))));
            }
            uint4 x = make_uint4(0, 0, 0, 0);
            if (row < n) {
                x = *reinterpret_cast<const uint4 *>(mats + ((size_t)2 * n + row) * grs + c);
                x = make_uint4(x.x ^ m[0], x.y ^ m[1], x.z ^ m[2], x.w ^ m[3]);
            }
            *reinterpret_cast<uint4 *>(D + at(row, c)) = x;
        }
        const int wpr = rs / 4;
        for (int i = t; i < nr * wpr; i += L) {
            const int row = i / wpr, c0 = (i - row * wpr) * 4;
            unsigned wg = 0;
            if (row < n) {
                const uint8_t *f = mats + (size_t)perm[row] * grs;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c0 + e < n) wg |= (unsigned)(f[perm[c0 + e]] ^ 0x80u) << (8 * e);
            }
            *reinterpret_cast<unsigned *>(G + at(row, c0)) = wg;
        }
    }
    block_sync();

    // ---- task waves: SD_u of their indices (both halves of the wave hold it); cost (Eq. 1)
    const bool task = wid < TW;
    int SDu[TC];
    if (task) {
        long long part = 0;
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            const int u = (wid * TC + c) * 32 + l5, uc = min(u, n - 1);
            int rd = 0, cd = 0, sg = 0, sd = 0;
            for (int k = 0; k < n; k += 16) {   // (entries past n are zero)
                const v4i x = lds16(G, at(uc, k)), y = lds16(D, at(uc, k));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    rd = __builtin_amdgcn_sdot4(x[e], y[e], rd, false);
                    sg = __builtin_amdgcn_sdot4(x[e], 0x01010101, sg, false);
                    sd = __builtin_amdgcn_sdot4(y[e], 0x01010101, sd, false);
                }
                if (!SYM) {
                    const int c0 = (wid * TC + c) * 32 + (lane & 16);
                    const v4i xc = cols16(G, k, c0), yc = cols16(D, k, c0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) cd = __builtin_amdgcn_sdot4(xc[e], yc[e], cd, false);
                }
            }
            SDu[c] = SYM ? 2 * rd : rd + cd;
            part += !half && u < n ? (long long)rd + 128LL * (sg + sd) + 16384LL * n : 0;
            if (!half && u < NP) rp[u] = SDu[c];   // for the blocks' first deltas
        }
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
        if (lane == 0) s_red[wid] = part;
    }
    int it = resume ? __builtin_amdgcn_readfirstlane(st->it) : 1;   // tabu: the iteration; 2opt: moves made + 1
    const int it_first = it;
    block_sync();
    long long cur = 0;
#pragma unroll
    for (int w = 0; w < TW; ++w) cur += s_red[w];
    auto uniform64 = [](long long x) -> long long {
        return ((long long)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) |
               (unsigned)__builtin_amdgcn_readfirstlane((int)x);
    };
    cur = uniform64(cur);
    long long best = resume ? uniform64(st->best) : cur;
    // cur - best, kept by every wave: the costs of two permutations differ by less than
    // n^2 255 * 127 < 2^31; cur and best themselves are the housekeeping wave's
    int gap = (int)(cur - best);
    const int cap = TABU ? a.iters : (a.iters > 0 ? a.iters : INT32_MAX - 1);

    // the next move, its pair and delta from sel (uniform); false when the search (or the
    // chunk) ends here
    int r = 0, s = 0, dstar = 0;
    bool improved = false, stopped = false;
    auto next_move = [&]() -> bool {
        const long long mk = sel[it & 1];
        if (RESUME && __builtin_amdgcn_readfirstlane(s_chunk_end)) return false;
        dstar = __builtin_amdgcn_readfirstlane((int)(mk >> 32));
        const int key = __builtin_amdgcn_readfirstlane((int)mk);
        if (TABU ? dstar == INT32_MAX : dstar >= 0) {
            stopped = true;
            return false;
        }
        r = key >> 9;
        s = key & 511;
        gap += dstar;
        improved = TABU && gap < 0;
        if (improved) gap = 0;
        return true;
    };
    // aspiration threshold of the next select: a tabu move is allowed below it
    auto aspire = [&]() -> int { return max(-gap, -(1 << 24)); };

    if (task) {
        // ================================================================ task waves
        const int crow = lane & 15, chunk = (lane >> 4) * 16;   // operand row and 16-byte column
        int uu[TC], ucl[TC], duu[TC], rowo[TC][2];
#pragma unroll
        for (int c = 0; c < TC; ++c) {
            uu[c] = (wid * TC + c) * 32 + l5;
            ucl[c] = min(uu[c], n - 1);
            duu[c] = D[at(ucl[c], ucl[c])];
#pragma unroll
            for (int h = 0; h < 2; ++h)   // operand rows: 16 indices each
                rowo[c][h] = at(min((wid * TC + c) * 32 + 16 * h + crow, n - 1), chunk);
        }
        const bool side_s = crow >= 8;     // operand rows 0..7 are side r, 8..15 side s
        const bool past = chunk + 64 * (KS - 1) >= n;   // the last step is past the rows
        const int colrow = min(chunk + 64 * (KS - 1), blk_rows(n) - 16);   // (there, stay inside)
        // D's operands do not change: kept in registers where those reach
        constexpr bool keep = TC == 1 && !BUSY && (SYM || KS <= 3);
        v4i drk[keep ? KS : 1][2], dck[keep && !SYM ? KS : 1][2];
        if constexpr (keep) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    drk[ks][h] = lds16(D, step(rowo[0][h], ks));
                    if (!SYM) dck[ks][h] = cols16(D, ks == KS - 1 ? colrow : chunk + 64 * ks, wid * 32 + 16 * h);
                }
        }
        int8_t *const M = half ? G : D;    // half 0 of the wave reads D, half 1 reads G
        int8_t *const sideM = side + half * 2 * 64 * KS;
        const int8_t *const sideA = side + (side_s ? 64 * KS : 0) + chunk;
        while (it <= cap) {
            block_sync();   // B1
            if (!next_move()) break;
            const int thr = aspire();
            // ---- A
            const int b = half ? s : r;
            const int mr = sx(r), ms = sx(s), offr = r * rs, offs = s * rs;
            // columns and rows r and s of D (half 0 of the wave) and G (half 1) at u
            int v0[TC], v1[TC], v2[TC], v3[TC];
#pragma unroll
            for (int c = 0; c < TC; ++c) {
                const int u = ucl[c], mu = sx(u);
                v2[c] = M[offr + (u ^ mr)];                                  // x_ru
                v3[c] = M[offs + (u ^ ms)];                                  // x_su
                v0[c] = SYM ? v2[c] : (int)M[u * rs + (r ^ mu)];             // x_ur
                v1[c] = SYM ? v3[c] : (int)M[u * rs + (s ^ mu)];             // x_us
            }
            const int dbb = D[at(b, b)];
            // the side rows of D, for B: their latency hides behind the differences
            const int so = at(side_s ? s : r, chunk);
            v4i sd[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) sd[ks] = lds16(D, step(so, ks));
            int dsum[TC], gsum[TC];
#pragma unroll
            for (int c = 0; c < TC; ++c) {
                const int u = uu[c];
                const bool valid = u < n, apart = u != r && u != s;
                const int pk = pack16(v0[c] - v1[c], v2[c] - v3[c]), sums = pack16(v0[c] + v2[c], v1[c] + v3[c]);
                // both halves get both: [0] from D, [1] from G
                const auto pp = __builtin_amdgcn_permlane32_swap(pk, pk, false, false);
                const auto ps = __builtin_amdgcn_permlane32_swap(sums, sums, false, false);
                const int dpk = (int)pp[0], gpk = (int)pp[1], dsm = (int)ps[0], gsm = (int)ps[1];
                // W_u, the index's share of the update in 8-bit limbs.  With x the pair of
                // differences of the wider matrix less 1 (in [-256, 254], two limbs) and y that
                // of the other (in [-127, 127]; minus 1 drops out of every difference), the
                // update of (u, v) is h_u + h_v - x_u.y_v - y_u.x_v, h = x.y = 128 M + L:
                //   half 0  [x limbs | -y twice | L | 1]   half 1  [-M in four limbs | -128 | 0 | 0]
                // and the operand of v is the same with each pair of words exchanged.
                const int xp = a.blk == 1 ? dpk : gpk, yp = a.blk == 1 ? gpk : dpk;
                const int x = pk_add(xp, -1), xa = pk_ashr<1>(x), xb = pk_sub(x, xa);
                const int X = bperm((unsigned)xb, (unsigned)xa, 0x06020400u);
                const int yn = pk_sub(0, yp), Y = bperm((unsigned)yn, (unsigned)yn, 0x02020000u);
                const int h = dot2(x, yp, 0), Mh = (h + 64) >> 7, Lh = h - (Mh << 7);
                const int mm = pack16(-Mh, -Mh);
                const int m01 = pk_ashr<2>(pk_add(mm, 0x00010000)), m23 = pk_ashr<2>(pk_add(mm, 0x00030002));
                const int H = bperm((unsigned)m23, (unsigned)m01, 0x06040200u);
                v4i w;
                w[0] = half ? H : X;
                w[1] = half ? (int)0x80808080 : Y;
                w[2] = half ? 0 : (Lh & 0xff);
                w[3] = half ? 0 : 1;
                if (valid) Wv[u * 2 + half] = w;
                if (half && valid && apart) {
                    const int mu = sx(u);
                    G[offr + (u ^ mr)] = (int8_t)v3[c];
                    G[offs + (u ^ ms)] = (int8_t)v2[c];
                    G[u * rs + (r ^ mu)] = (int8_t)v1[c];
                    G[u * rs + (s ^ mu)] = (int8_t)v0[c];
                }
                if (!SYM && valid && (!half || apart)) {
                    sideM[u] = (int8_t)(half ? v1[c] : v0[c]);
                    sideM[64 * KS + u] = (int8_t)(half ? v0[c] : v1[c]);
                }
                SDu[c] -= dot2(dpk, gpk, 0);
                dsum[c] = (half ? dsm >> 16 : (int)(short)dsm) - duu[c] - dbb;   // d_ub + d_bu - d_uu - d_bb
                gsum[c] = half ? (int)(short)gsm : gsm >> 16;                    // g_ub + g_bu under p'
            }
            block_sync();   // B2
            // ---- B: C[b][u] = T'_ub + T'_bu, and SD'_r, SD'_s
            const int gbb = G[at(b, b)];
            int guu[TC];
            unsigned tb[TC];
#pragma unroll
            for (int c = 0; c < TC; ++c) {
                guu[c] = G[at(ucl[c], ucl[c])];
                if (marks)
                    tb[c] = mark[ucl[c]] > it + 1 || mark[b] > it + 1 ? ~0u : 0u;
                else
                    tb[c] = TABU && wid * TC + c < NB ? bits[b * NB + wid * TC + c] : 0u;
            }
            asm volatile("" ::: "memory");   // those first: they come back with the rows below
            v4i cc[TC][2], cs = {0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < TC; ++c) cc[c][0] = cc[c][1] = v4i{0, 0, 0, 0};
            // A step's operands are asked for together, then consumed: left to itself the
            // compiler keeps about two reads in flight, and a task wave waits out an LDS round
            // trip per product (BUSY kernels have no registers for it, and other searches to
            // run meanwhile)
            auto together = [] {
                if constexpr (!BUSY) __builtin_amdgcn_sched_barrier(0);
            };
            constexpr bool both = TC == 1 && !BUSY;   // rows and columns in one go
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                v4i sdr_ = sd[ks], sgr_ = lds16(G, step(so, ks)), sdc, sgc;
                v4i gr[TC][2], dr[TC][2], gc[TC][2], dc[TC][2];
#pragma unroll
                for (int c = 0; c < TC; ++c)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        gr[c][h] = lds16(G, step(rowo[c][h], ks));
                        dr[c][h] = keep ? drk[keep ? ks : 0][h] : lds16(D, step(rowo[c][h], ks));
                    }
                // the same along the columns (zero past n in the side buffers)
                auto load_columns = [&] {
                    sdc = lds16(sideA, 64 * ks);
                    sgc = lds16(sideA, 2 * 64 * KS + 64 * ks);
                    const int k = ks == KS - 1 ? colrow : chunk + 64 * ks;
#pragma unroll
                    for (int c = 0; c < TC; ++c)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int c0 = (wid * TC + c) * 32 + 16 * h;
                            gc[c][h] = cols16(G, k, c0);
                            dc[c][h] = keep ? dck[keep && !SYM ? ks : 0][h] : cols16(D, k, c0);
                        }
                };
                if (!SYM && both) load_columns();
                together();
                if (ks == KS - 1 && past) {
                    sdr_ = v4i{0, 0, 0, 0};   // past the row: whatever the rows hold there
                    sgr_ = v4i{0, 0, 0, 0};
                }
                cs = __builtin_amdgcn_mfma_i32_16x16x64_i8(sdr_, sgr_, cs, 0, 0, 0);
#pragma unroll
                for (int c = 0; c < TC; ++c)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        cc[c][h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sdr_, gr[c][h], cc[c][h], 0, 0, 0);
                        cc[c][h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sgr_, dr[c][h], cc[c][h], 0, 0, 0);
                    }
                if constexpr (!SYM) {
                    if (!both) {
                        load_columns();
                        together();
                    }
                    cs = __builtin_amdgcn_mfma_i32_16x16x64_i8(sdc, sgc, cs, 0, 0, 0);
#pragma unroll
                    for (int c = 0; c < TC; ++c)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            cc[c][h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sdc, gc[c][h], cc[c][h], 0, 0, 0);
                            cc[c][h] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sgc, dc[c][h], cc[c][h], 0, 0, 0);
                        }
                }
            }
            const int sdr = __builtin_amdgcn_readlane(cs[0], 0), sds = __builtin_amdgcn_readlane(cs[0], 63);
            const int SDr = SYM ? 2 * sdr : sdr, SDs = SYM ? 2 * sds : sds;
            int d = INT32_MAX, key = KEY_NONE;
#pragma unroll
            for (int c = 0; c < TC; ++c) {
                const int u = uu[c];
                const int cv = ((lane >> 4) & 1) ? cc[c][1][0] : cc[c][0][0];
                if (u == r) SDu[c] = SDr;
                if (u == s) SDu[c] = SDs;
                int dl = (SYM ? 2 * cv : cv) - SDu[c] - (half ? SDs : SDr) + __mul24(dsum[c], gsum[c] - guu[c] - gbb);
                if (u == r || u == s) dl = -dstar;       // the move undone
                const bool real = u < n && u != b;
                const bool tabu = TABU && ((tb[c] >> l5) & 1u);
                if (TC * TW == NB || u < NP) rp[half * NP + u] = !real ? BK_NOMOVE : (tabu && !marks ? dl + BK_OFF : dl - BK_OFF);
                const bool adm = real && (!tabu || dl < thr);
                const int dc = adm ? dl : INT32_MAX, kc = (min(u, b) << 9) | max(u, b);
                if (c == 0) {
                    d = dc;
                    key = kc;
                } else {
                    const bool take = dc < d || (dc == d && kc < key);
                    d = take ? dc : d;
                    key = take ? kc : key;
                }
            }
            const int wd = wmin32(d);
            if (wd != INT32_MAX) {
                const unsigned long long tie = __ballot(d == wd);
                int wk;
                if (__builtin_popcountll(tie) == 1)
                    wk = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(tie));
                else
                    wk = wmin32(d == wd ? key : KEY_NONE);
                if (lane == 0) sel_min(&sel[(it + 1) & 1], wd, wk);
            }
            ++it;
        }
    } else if (wid == TW) {
        // ======================================================= housekeeping wave
        int myev = -1;
        // pairs whose latest tenure ends at iteration x, among moves up to `last`
        auto find_events = [&](int x, int last) {
            const int tn = lo + lane, i = x - tn;
            myev = -1;
            if (tn <= hi && i <= last) {
                const int e = ring[i & rmask];
                if ((e >> 18) == tn) myev = e & 0x3ffff;
            }
            const unsigned long long m = __ballot(myev >= 0);
            const int c = __builtin_popcountll(m);
            if (myev >= 0) s_ev[1 + __builtin_popcountll(m & ((1ull << lane) - 1))] = myev;
            if (lane == 0) s_ev[0] = c;
        };
        if (TABU && !marks) find_events(it + 1, it - 1);
        // tenures of iterations it .. it + 63 (lane i: it + i), and the next ones in the making
        Tenures next;
        int tens = 0, tpos = 0;
        if (TABU) {
            next.begin(a.seed, (long long)it + lane, a.start_id);
#pragma unroll 1
            for (int i = 0; i < 10; ++i) next.round();
            tens = next.value(lo, hi);
            next.begin(a.seed, (long long)it + 64 + lane, a.start_id);
        }
        const long long clock_end = RESUME && a.budget > 0 ? (long long)wall_clock64() + a.budget : 0;
        while (it <= cap) {
            const int tn = TABU ? __builtin_amdgcn_readlane(tens, tpos) : 0;
            // chunk end: decided every 16 iterations, read by every wave after B1
            if (RESUME && clock_end != 0 && it != it_first && (it & 15) == 0 && lane == 0)
                s_chunk_end = (long long)wall_clock64() >= clock_end;
            block_sync();   // B1
            if (!next_move()) break;
            cur += dstar;
            // ---- A
            if (lane == 0) sel[(it + 1) & 1] = BK_NONE;
            const unsigned was = TABU && !marks ? bits[r * NB + (s >> 5)] : 0u;
            if (lane < 4) {    // the corners of G: (r, r), (r, s), (s, r), (s, s) take (sigma, sigma)
                const int i = lane & 2 ? s : r, j = lane & 1 ? s : r;
                const int si = lane & 2 ? r : s, sj = lane & 1 ? r : s;
                const int8_t x = G[at(si, sj)];
                G[at(i, j)] = x;
                if (!SYM) side[(lane & 1 ? 3 : 2) * 64 * KS + i] = x;
            }
            if (improved) {
                best = cur;
                for (int x = lane; x < n; x += 64) bestp[x] = perm[x == r ? s : (x == s ? r : x)];
            }
            if (FREQ && lane == 0)
                __hip_atomic_fetch_add(a.freq + pidx(n, r, s), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (marks) {   // the two units moved now sit at s and r
                if (lane < 2) mark[lane ? s : r] = it + tn;
            } else if (TABU) {
                const int pr = (r << 9) | s;
                if (myev >= 0) {
                    const int x = myev >> 9, y = myev & 511;
                    atomicAnd(&bits[x * NB + (y >> 5)], ~(1u << (y & 31)));
                    atomicAnd(&bits[y * NB + (x >> 5)], ~(1u << (x & 31)));
                }
                // tabu and not about to expire (made by aspiration): its older entry is void
                if (((__builtin_amdgcn_readfirstlane((int)was) >> (s & 31)) & 1) && __ballot(myev == pr) == 0)
                    for (int x = lane; x <= rmask; x += 64) {
                        const int e = ring[x];
                        if (e >= 0 && (e & 0x3ffff) == pr) ring[x] = -1;
                    }
                if (lane < 2) {
                    if (lane == 0) ring[it & rmask] = (tn << 18) | pr;
                    const int x = lane ? s : r, y = lane ? r : s;
                    // tabu at it + 1 from a tenure of 2 on
                    if (tn >= 2)
                        atomicOr(&bits[x * NB + (y >> 5)], 1u << (y & 31));
                    else
                        atomicAnd(&bits[x * NB + (y >> 5)], ~(1u << (y & 31)));
                }
            }
            block_sync();   // B2
            // ---- B
            if (lane == 0) {
                const int x = perm[r], y = perm[s];
                perm[r] = y;
                perm[s] = x;
            }
            if (TABU) {
                if (!marks) find_events(it + 2, it);
                if (tpos < 10) next.round();
                if (++tpos == 64) {
                    tpos = 0;
                    tens = next.value(lo, hi);
                    next.begin(a.seed, (long long)it + 65 + lane, a.start_id);
                }
            }
            ++it;
        }
    } else {
        // ================================================================ block waves
        int bI[BPW], bJ[BPW];
        const int first = (wid - TW - 1) * BPW, cnt = min(BPW, SH::NBLK - first);
#pragma unroll
        for (int q = 0; q < BPW; ++q) {
            int id = min(first + q, SH::NBLK - 1), i = 0;
            while (id >= NB - i) {
                id -= NB - i;
                ++i;
            }
            bI[q] = i;
            bJ[q] = i + id;
        }
        const auto has = [&](int q) -> bool { return q == 0 || q < cnt; };
        // the wave's blocks in a row or column of blocks, as a mask of q (four bits each): one
        // test passes over those a move does not touch
        static_assert(BPW <= 4, "four bits");
        unsigned long long tabI = 0, tabJ = 0;
#pragma unroll
        for (int q = 0; q < BPW; ++q)
            if (has(q)) {
                tabI |= 1ull << (4 * bI[q] + q);
                tabJ |= 1ull << (4 * bJ[q] + q);
            }
        auto in_row = [&](int x) -> unsigned {
            if constexpr (BPW == 1) return bI[0] == (x >> 5) ? 1u : 0u;
            return (unsigned)(tabI >> (4 * (x >> 5))) & 15u;
        };
        auto in_col = [&](int x) -> unsigned {
            if constexpr (BPW == 1) return bJ[0] == (x >> 5) ? 1u : 0u;
            return (unsigned)(tabJ >> (4 * (x >> 5))) & 15u;
        };
        v16i acc[BPW];
#pragma unroll
        for (int q = 0; q < BPW; ++q) {
            if (!has(q)) continue;
            const int v = bJ[q] * 32 + l5, vc = min(v, n - 1);
            if (resume || a.table) {
                // the saved slots of the chunk before, or the caller's neighbourhood of the start
                const int32_t *const src = resume ? a.st_slots : a.table;
                const int off = resume ? 0 : BK_OFF;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int x = bI[q] * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
                    const bool real = x < n && v < n && x != v;
                    acc[q][i] = real ? src[pidx(n, min(x, v), max(x, v))] - off : BK_NOMOVE;
                    if (RESUME && real && x < v && acc[q][i] > 0) {   // tabu
                        atomicOr(&bits[x * NB + (v >> 5)], 1u << (v & 31));
                        atomicOr(&bits[v * NB + (x >> 5)], 1u << (x & 31));
                    }
                }
                continue;
            }
            // ---- first deltas: T_ij + T_ji by the contraction, then the rest of Eq. (2)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[q][i] = 0;
            const int xr = min(bI[q] * 32 + l5, n - 1);
            for (int k = 0; k < n; k += 32) {
                const int kk = k + half * 16;
                const bool in = kk < n;
                const int kc = min(kk, blk_rows(n) - 16);
                v4i gi = lds16(G, at(xr, kc)), di = lds16(D, at(xr, kc));
                v4i gj = lds16(G, at(vc, kc)), dj = lds16(D, at(vc, kc));
                if (!in) gi = di = v4i{0, 0, 0, 0};
                acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gi, dj, acc[q], 0, 0, 0);
                acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(di, gj, acc[q], 0, 0, 0);
                if constexpr (!SYM) {
                    const int ci = bI[q] * 32 + (lane & 16), cj = bJ[q] * 32 + (lane & 16);
                    gi = cols16(G, kc, ci), di = cols16(D, kc, ci);
                    gj = cols16(G, kc, cj), dj = cols16(D, kc, cj);
                    if (!in) gi = di = v4i{0, 0, 0, 0};
                    acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gi, dj, acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(di, gj, acc[q], 0, 0, 0);
                }
            }
            const int dvv = D[at(vc, vc)], gvv = G[at(vc, vc)], sdv = rp[v];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int x = bI[q] * 32 + 8 * (i >> 2) + 4 * half + (i & 3), xc = min(x, n - 1);
                const int ds = (int)D[at(xc, vc)] + (int)D[at(vc, xc)] - (int)D[at(xc, xc)] - dvv;
                const int gs = (int)G[at(xc, vc)] + (int)G[at(vc, xc)] - (int)G[at(xc, xc)] - gvv;
                const int full = (SYM ? 2 * acc[q][i] : acc[q][i]) - rp[x] - sdv + __mul24(ds, gs);
                acc[q][i] = x < n && v < n && x != v ? full - BK_OFF : BK_NOMOVE;
            }
        }
        // candidate of the wave's blocks for iteration x into sel, columns er and es left out
        auto candidates = [&](int er, int es, int x, int thr) {
            const int thrk = (thr - BK_OFF) * 32;
            int cand = INT32_MAX, base = (bI[0] << 14) | (bJ[0] << 5);   // of the candidate's block
#pragma unroll
            for (int q = 0; q < BPW; ++q) {
                if (!has(q)) break;
                int k[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) k[i] = acc[q][i] * 32 + (8 * (i >> 2) + (i & 3));
                int lo_ = min(k[0], k[1]);
                unsigned um = min((unsigned)k[0], (unsigned)k[1]);
#pragma unroll
                for (int i = 2; i < 16; i += 2) {
                    lo_ = min(min(lo_, k[i]), k[i + 1]);
                    if (TABU) um = min(min(um, (unsigned)k[i]), (unsigned)k[i + 1]);
                }
                int c = lo_;
                if (marks) {
                    // every slot is held as free: the lowest of all where it is below the
                    // threshold, else the lowest with neither unit marked
                    int f = INT32_MAX;
#pragma unroll
                    for (int y = 0; y < 4; ++y) {
                        const v4i mr = *reinterpret_cast<const v4i *>(mark + bI[q] * 32 + 8 * y + 4 * half);
#pragma unroll
                        for (int e = 0; e < 4; ++e) f = min(f, mr[e] > x ? INT32_MAX : k[4 * y + e]);
                    }
                    if (mark[bJ[q] * 32 + l5] > x) f = INT32_MAX;
                    c = lo_ < thrk ? lo_ : f;
                } else if (TABU) {
                    const int ta = (int)(um ^ 0x80000000u);   // the lowest tabu slot, as if free
                    c = ta < thrk ? min(lo_, ta) : lo_;
                }
                c |= half << 2;
                const int v = bJ[q] * 32 + l5;
                c = v == er || v == es ? INT32_MAX : c;
                if (q == 0) {
                    cand = c;
                } else {
                    // blocks come in order of I, then J: between equal deltas of one row of
                    // blocks the lower row wins, then the earlier block, and across them the
                    // earlier row of blocks (whose row bits move to base, so that it does)
                    const int m = bI[q] == bI[q - 1] ? 0 : 31;
                    base += (cand & m) << 9;
                    cand &= ~m;
                    const bool take = c < cand;
                    cand = take ? c : cand;
                    base = take ? (bI[q] << 14) | (bJ[q] << 5) : base;
                }
            }
            if constexpr (BPW == 1) {
                const int wm = wmin32(cand);
                if (wm < 0) {   // lanes that tie hold the same row: the lowest column
                    const int ln = (int)__builtin_ctzll(__ballot(cand == wm));
                    if (lane == 0) sel_min(&sel[x & 1], (wm >> 5) + BK_OFF, base + ((wm & 31) << 9) + (ln & 31));
                }
            } else {
                const int d = cand >> 5, wd = wmin32(d), key = base + ((cand & 31) << 9) + l5;
                if (wd < 0) {
                    const unsigned long long tie = __ballot(d == wd);
                    const int wk = __builtin_popcountll(tie) == 1
                                       ? __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(tie))
                                       : wmin32(d == wd ? key : KEY_NONE);
                    if (lane == 0) sel_min(&sel[x & 1], wd + BK_OFF, wk);
                }
            }
        };
        // the value of row x in block q of the wave
        auto set_row = [&](int q, int x, int val) {
            const int i = ((x >> 3) & 3) * 4 + (x & 3), old = acc[q][i];
            acc[q][i] = half == ((x >> 2) & 1) ? val : old;
        };
        constexpr int NOWHERE = 8 * 32;       // an index in no block
        int r0 = NOWHERE, s0 = NOWHERE;       // the move before: its rows and columns are stale
        int rowv[BPW][2];                     // the deltas recomputed for its rows
        auto patch = [&]() {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int x = h ? s0 : r0;
                const unsigned mi = in_row(x), mj = in_col(x);
                if (mi) {
                    stay_branch();
#pragma unroll
                    for (int q = 0; q < BPW; ++q)
                        if (BPW == 1 || (mi >> q) & 1) {
                            stay_branch();
                            set_row(q, x, rowv[q][h]);
                        }
                }
                if (mj) {
                    stay_branch();
#pragma unroll
                    for (int q = 0; q < BPW; ++q)
                        if (BPW == 1 || (mj >> q) & 1) {
                            stay_branch();
                            const bool mine = l5 == (x & 31);
                            v4i val[4];
#pragma unroll
                            for (int y = 0; y < 4; ++y)
                                val[y] = *reinterpret_cast<const v4i *>(rp + h * NP + bI[q] * 32 + 8 * y + 4 * half);
#pragma unroll
                            for (int y = 0; y < 4; ++y)
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[q][4 * y + e] = mine ? val[y][e] : acc[q][4 * y + e];
                        }
                }
            }
        };
        candidates(-1, -1, it, aspire());
        while (it <= cap) {
            block_sync();   // B1
            // what A needs beside the move, read together with it
#pragma unroll
            for (int q = 0; q < BPW; ++q)
                if (has(q)) {
                    rowv[q][0] = rp[bJ[q] * 32 + l5];
                    rowv[q][1] = rp[NP + bJ[q] * 32 + l5];
                }
            v4i ev = {0, 0, 0, 0};
            if (TABU) ev = *reinterpret_cast<const v4i *>(s_ev);
            if (!next_move()) break;
            const int thr = aspire();
            // ---- A
            patch();
            if (TABU) {
                const int nev = __builtin_amdgcn_readfirstlane(ev[0]);
                for (int e = 0; e < nev; ++e) {
                    const int pr = __builtin_amdgcn_readfirstlane(e == 0 ? ev[1] : (e == 1 ? ev[2] : s_ev[1 + e]));
                    const int x = pr >> 9, y = pr & 511;
                    const unsigned me = in_row(x) & in_col(y);
                    if (me == 0) continue;
                    stay_branch();
#pragma unroll
                    for (int q = 0; q < BPW; ++q)
                        if (BPW == 1 || (me >> q) & 1) {
                            stay_branch();
                            const int i = ((x >> 3) & 3) * 4 + (x & 3), old = acc[q][i];
                            acc[q][i] = half == ((x >> 2) & 1) && l5 == (y & 31) ? old - 2 * BK_OFF : old;
                            if (bI[q] == bJ[q]) {   // the mirror slot of a diagonal block
                                stay_branch();
                                const int j = ((y >> 3) & 3) * 4 + (y & 3), ol2 = acc[q][j];
                                acc[q][j] = half == ((y >> 2) & 1) && l5 == (x & 31) ? ol2 - 2 * BK_OFF : ol2;
                            }
                        }
                }
            }
            // rows r and s are the task waves' until the next A: out of the minimum (the
            // update moves these slots by less than 2^19, which leaves them above every key)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int x = h ? s : r;
                const unsigned mi = in_row(x);
                if (mi == 0) continue;
                stay_branch();
#pragma unroll
                for (int q = 0; q < BPW; ++q)
                    if (BPW == 1 || (mi >> q) & 1) {
                        stay_branch();
                        set_row(q, x, BK_NOMOVE - (1 << 20));
                    }
            }
            block_sync();   // B2
            // ---- B (its few reads go before the task waves' many)
            __builtin_amdgcn_s_setprio(3);
#pragma unroll
            for (int q = 0; q < BPW; ++q) {
                if (!has(q)) break;
                const v4i wa = Wv[(bI[q] * 32 + l5) * 2 + half], wb = Wv[(bJ[q] * 32 + l5) * 2 + half];
                const v4i wx = {wb[1], wb[0], wb[3], wb[2]};
                acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa, wx, acc[q], 0, 0, 0);
            }
            __builtin_amdgcn_s_setprio(0);
            candidates(r, s, it + 1, thr);
            r0 = r;
            s0 = s;
            ++it;
        }
        if (RESUME && !stopped && it <= cap) {   // the chunk ends: save the slots, nothing stale
            patch();                             // (B1 of this iteration was passed)
#pragma unroll
            for (int q = 0; q < BPW; ++q) {
                if (!has(q)) break;
                const int v = bJ[q] * 32 + l5;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int x = bI[q] * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
                    if (x < v && v < n) a.st_slots[pidx(n, x, v)] = acc[q][i];
                }
            }
        }
    }

    // ---- results
    block_sync();
    const bool finished = !RESUME || stopped || it > cap;
    if (RESUME) {
        for (int x = t; x < n; x += L) {
            a.st_perm[x] = perm[x];
            a.st_bestp[x] = bestp[x];
        }
        if (!finished)
            for (int x = t; x <= rmask; x += L) a.st_ring[x] = ring[x];
        if (t == TW * 64) {
            st->cur = cur;
            st->best = best;
            st->it = it;
            st->moves = it - 1;
            st->done = finished ? 1 : 0;
        }
        if (!finished) return;
    }
    const int *const res = TABU ? bestp : perm;
    for (int x = t; x < n; x += L) a.perm_out[x] = res[x];
    if (t == TW * 64) {
        *a.cost_out = TABU ? best : cur;
        if (a.steps_out) *a.steps_out = it - 1;
    }
}

// Block b runs items[b] of a batch, or search job0 + b of a launch on one instance.  BUSY
// (NB <= 4): held to 64 VGPRs, so that two and more searches share a compute unit, for
// launches of more searches than compute units; else a task wave keeps more of its
// operands in flight.
template <int NB, bool SYM, bool TABU, bool BUSY, bool FREQ>
__global__ void __launch_bounds__(Shape<NB>::LANES) __attribute__((amdgpu_waves_per_eu(BUSY ? 8 : 4)))
block_kernel(SearchArgs a, BatchArgs b) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ __align__(16) BlkShared sh;
    Item it{};
    if (b.items) {
        it = b.items[blockIdx.x];
        it.perm_in = b.perms + it.perm_off;
        it.perm_out = b.perms + it.perm_off;
        it.cost_out = b.best + it.out_off;
        it.steps_out = b.done ? b.done + it.out_off : nullptr;
    } else {
        const int job = a.job0 + blockIdx.x;
        it.mats = a.mats;
        it.table = a.table ? a.table + (size_t)job * a.m : nullptr;
        it.perm_in = a.perms_in + (size_t)job * a.n;
        it.perm_out = a.perm_out + (size_t)job * a.n;
        it.cost_out = a.cost_out + job;
        it.steps_out = a.steps_out ? a.steps_out + job : nullptr;
        it.n = a.n;
        it.iters = a.iters;
        it.lo = a.lo;
        it.hi = a.hi;
        it.seed = a.seed;
        it.start_id = a.start_base + job;
        it.blk = a.blk;
        if (FREQ) {
            it.m = a.m;
            it.freq = a.freq + (size_t)job * a.m;
            it.attr = a.attr;
        }
    }
    block_body<NB, SYM, TABU, false, BUSY, FREQ>(it, sm, sh);
}

template <int NB, bool SYM, bool TABU, bool BUSY, bool FREQ>
hipError_t launch_nb(const SearchArgs &a, const BatchArgs &b, int grid, size_t smem, hipStream_t st) {
    hipLaunchKernelGGL((block_kernel<NB, SYM, TABU, BUSY, FREQ>), dim3(grid), dim3(Shape<NB>::LANES), smem, st, a, b);
    return report(hipGetLastError(), "block kernel launch");
}

template <bool TABU, bool BUSY, bool FREQ = false>
hipError_t launch_any(int form, const SearchArgs &a, const BatchArgs &b, int grid, size_t smem, hipStream_t st) {
    switch (form) {
        case 0: return launch_nb<1, false, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 1: return launch_nb<1, true, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 2: return launch_nb<2, false, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 3: return launch_nb<2, true, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 4: return launch_nb<3, false, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 5: return launch_nb<3, true, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 6: return launch_nb<4, false, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        case 7: return launch_nb<4, true, TABU, BUSY, FREQ>(a, b, grid, smem, st);
        default: break;
    }
    if constexpr (!BUSY)
        switch (form) {
            case 8: return launch_nb<5, false, TABU, false, FREQ>(a, b, grid, smem, st);
            case 9: return launch_nb<5, true, TABU, false, FREQ>(a, b, grid, smem, st);
            case 10: return launch_nb<6, false, TABU, false, FREQ>(a, b, grid, smem, st);
            case 11: return launch_nb<6, true, TABU, false, FREQ>(a, b, grid, smem, st);
            case 12: return launch_nb<7, false, TABU, false, FREQ>(a, b, grid, smem, st);
            case 13: return launch_nb<7, true, TABU, false, FREQ>(a, b, grid, smem, st);
            case 14: return launch_nb<8, false, TABU, false, FREQ>(a, b, grid, smem, st);
            case 15: return launch_nb<8, true, TABU, false, FREQ>(a, b, grid, smem, st);
            default: break;
        }
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace qapk
