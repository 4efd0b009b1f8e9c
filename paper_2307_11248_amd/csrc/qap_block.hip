// qap_block.hip -- block form of the tabu and 2opt searches: one workgroup per search, the
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
//   * the recomputed deltas of rows r and s are a contraction too: a task wave takes 32
//     indices u and gets Delta(u, r), Delta(u, s) from v_mfma_i32_16x16x64_i8 on the rows
//     of G, G^T, D, D^T against the eight side rows, with one correction product each;
//   * the tabu state of a slot is an offset in its value, so the select of a block is a
//     signed minimum (the free slots) and an unsigned minimum (the tabu ones) of the
//     same keys, with no test per slot.
//
// Waves.  NB = ceil(n / 32).  NB task waves (32 indices x the two sides r, s: one pair a
// lane), one housekeeping wave, and the block waves, BPW blocks (I <= J) each.
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
//   A       task waves  bytes of columns r and s of D and G for their u; W_u; G and G^T
//                       follow the move (rows and columns r, s exchanged in place)
//           block waves the rows and columns of the move before this one take the deltas
//                       the task waves recomputed then; tabu moves that expire are freed
//           housekeeping the corner entries of G; tabu bits and ring; best-so-far
//   B2
//   B       task waves  Delta'(u, r), Delta'(u, s) under p', their candidate for it + 1
//           block waves one MFMA a block, candidate of every slot outside r and s
//           housekeeping p; the tabu moves that expire at it + 2
// The rows and columns of r and s in the blocks are stale between B and the next A and are
// left out of the blocks' minimum; the task waves' candidates stand for them.
#include "qap_internal.h"

namespace qapk {

namespace {

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
    static constexpr int NBLK = NB * (NB + 1) / 2;
    // blocks per block wave: one while the workgroup fits 16 waves
    static constexpr int BPW = NB <= 4 ? 1 : (NB == 5 ? 2 : (NB == 6 ? 3 : (NB == 7 ? 4 : 6)));
    static constexpr int BW = (NBLK + BPW - 1) / BPW;
    static constexpr int TW = NB;                     // task waves
    static constexpr int WAVES = TW + 1 + BW;
    static constexpr int LANES = WAVES * 64;
    static constexpr int KS = (NB + 1) / 2;           // 64-byte steps of a row
};

// LDS row stride: an odd multiple of 16 bytes, so 16 consecutive rows start in 16 different
// 16-byte columns of the banks.
__host__ __device__ inline int blk_stride(int n) { return (((n + 15) / 16) | 1) * 16; }

struct BlkPlan {
    int g, gt, d, dt, w, rp, perm, bestp, bits, ring, ten, total;
};

__host__ __device__ inline int blk_ring(int hi) {
    int r = 32;
    while (r < hi + 2) r *= 2;
    return r;
}

__host__ __device__ inline BlkPlan blk_plan(int n, int nb, int lanes, int sym, int hi, bool tabu) {
    const int rs = blk_stride(n), np = nb * 32;
    BlkPlan q;
    int o = 0;
    auto take = [&o](int bytes) { int at = o; o += (bytes + 15) & ~15; return at; };
    q.g = take(n * rs);
    q.gt = sym ? q.g : take(n * rs);
    q.d = take(n * rs);
    q.dt = sym ? q.d : take(n * rs);
    q.w = take(np * 32);      // also what a row's last 64-byte step may read past the matrices
    q.rp = take(np * 2 * 4);
    q.perm = take(np * 4);
    q.bestp = take(np * 4);
    q.bits = take(tabu ? np * nb * 4 : 0);
    q.ring = take(tabu ? blk_ring(hi) * 4 : 0);
    q.ten = take(tabu ? lanes * 4 : 0);
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

// Philox4x64-10 (Salmon et al., SC'11), first output word; the tenure of the move of
// iteration `it` of start `start` (Sec. 4.3): uniform in [lo, hi].
__device__ inline int blk_tenure(unsigned long long seed, long long it, long long start, int lo, int hi) {
    const unsigned long long M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    const unsigned long long W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
    unsigned long long c0 = (unsigned long long)it, c1 = (unsigned long long)start, c2 = 0, c3 = 0, k0 = seed, k1 = 0;
#pragma unroll 1
    for (int round = 0; round < 10; ++round) {
        if (round > 0) { k0 += W0; k1 += W1; }
        const unsigned long long hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        const unsigned long long hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        const unsigned long long n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    }
    const unsigned long long span = (unsigned long long)((long long)hi - lo + 1);
    return lo + (int)(((c0 >> 32) * span) >> 32);
}

__device__ inline void sel_min(long long *slot, int d, int key) {
    __hip_atomic_fetch_min(slot, ((long long)d << 32) | (unsigned)key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int NB, bool SYM, bool TABU>
__device__ __attribute__((always_inline)) void block_body(const Item &a, unsigned char *sm) {
    using SH = Shape<NB>;
    constexpr int KS = SH::KS, L = SH::LANES, TW = SH::TW, BPW = SH::BPW, NP = NB * 32;
    constexpr int NM = SYM ? 1 : 2;   // matrices of a kind (with their transposes)
    __shared__ int s_bad;
    __shared__ long long sel[2];
    __shared__ long long s_red[TW];
    __shared__ int s_ev[68];          // count, then the pairs that become free
    const int n = a.n, rs = blk_stride(n), t = threadIdx.x, lane = t & 63;
    const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
    const int half = lane >> 5, l5 = lane & 31;
    const int hi = TABU ? a.hi : 0, lo = TABU ? a.lo : 0;
    const BlkPlan P = blk_plan(n, NB, L, SYM, hi, TABU);
    const int rmask = blk_ring(hi) - 1;
    int8_t *const smb = reinterpret_cast<int8_t *>(sm);
    int8_t *const G = smb + P.g, *const GT = smb + P.gt, *const D = smb + P.d, *const DT = smb + P.dt;
    v4i *const Wv = reinterpret_cast<v4i *>(sm + P.w);   // two 16-byte halves per index
    int *const rp = reinterpret_cast<int *>(sm + P.rp);
    int *const perm = reinterpret_cast<int *>(sm + P.perm), *const bestp = reinterpret_cast<int *>(sm + P.bestp);
    unsigned *const bits = reinterpret_cast<unsigned *>(sm + P.bits);
    int *const ring = reinterpret_cast<int *>(sm + P.ring), *const ten = reinterpret_cast<int *>(sm + P.ten);

    // ---- read and check the start
    if (t == 0) s_bad = 0;
    for (int u = t; u < NP; u += L) rp[u] = -1;
    for (int i = t; i < NP * 8; i += L) reinterpret_cast<int *>(Wv)[i] = 0;
    if (TABU) {
        for (int i = t; i < NP * NB; i += L) bits[i] = 0;
        for (int i = t; i <= rmask; i += L) ring[i] = -1;
    }
    if (t < 2) sel[t] = BK_NONE;
    __syncthreads();
    for (int u = t; u < n; u += L) {
        const int v = a.perm_in[u];
        perm[u] = v;
        bestp[u] = v;
        if (v < 0 || v >= n || atomicExch(&rp[v], u) != -1) s_bad = 1;
    }
    __syncthreads();
    if (s_bad) {
        if (a.perm_out != a.perm_in)
            for (int u = t; u < n; u += L) a.perm_out[u] = a.perm_in[u];
        if (t == 0) {
            *a.cost_out = INT64_MIN;
            if (a.steps_out) *a.steps_out = -2;  // QAP_E_NOT_PERM
        }
        return;
    }

    // ---- stage D, D^T and gather G = F[p][p], G^T (entries minus 128, zero past n)
    {
        const int grs = row_stride(n), vpr = rs / 16;
        const uint8_t *const mats = a.mats;
        for (int i = t; i < n * vpr; i += L) {
            const int row = i / vpr, c = (i - row * vpr) * 16;
            unsigned m[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int real = n - (c + 4 * e);
                m[e] = real >= 4 ? 0x80808080u : (real <= 0 ? 0u : (0x80808080u >> (8 * (4 - real))));
            }
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const uint4 x = *reinterpret_cast<const uint4 *>(mats + ((size_t)(2 + q) * n + row) * grs + c);
                *reinterpret_cast<uint4 *>((q ? DT : D) + row * rs + c) =
                    make_uint4(x.x ^ m[0], x.y ^ m[1], x.z ^ m[2], x.w ^ m[3]);
            }
        }
        const int wpr = rs / 4;
        for (int i = t; i < n * wpr; i += L) {
            const int row = i / wpr, c0 = (i - row * wpr) * 4;
            const uint8_t *f = mats + (size_t)perm[row] * grs;
            unsigned wg = 0, wgt = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c0 + e < n) {
                    const int pc = perm[c0 + e];
                    wg |= (unsigned)(f[pc] ^ 0x80u) << (8 * e);
                    if (!SYM) wgt |= (unsigned)(f[(size_t)n * grs + pc] ^ 0x80u) << (8 * e);
                }
            reinterpret_cast<unsigned *>(G)[i] = wg;
            if (!SYM) reinterpret_cast<unsigned *>(GT)[i] = wgt;
        }
    }
    __syncthreads();

    // ---- task waves: SD_u of their index (both halves of the wave hold it); cost (Eq. 1)
    const bool task = wid < TW;
    const int u = wid * 32 + l5, uc = min(u, n - 1);   // (task waves)
    int SDu = 0;
    if (task) {
        const int8_t *x = (half && !SYM ? GT : G) + uc * rs, *y = (half && !SYM ? DT : D) + uc * rs;
        int dot = 0, sx = 0, sy = 0;
        for (int k = 0; k < n; k += 4) {   // (bytes past n are zero)
            const int xw = *reinterpret_cast<const int *>(x + k), yw = *reinterpret_cast<const int *>(y + k);
            dot = __builtin_amdgcn_sdot4(xw, yw, dot, false);
            sx = __builtin_amdgcn_sdot4(xw, 0x01010101, sx, false);
            sy = __builtin_amdgcn_sdot4(yw, 0x01010101, sy, false);
        }
        SDu = dot + __shfl_xor(dot, 32, 64);
        long long part = !half && u < n ? (long long)dot + 128LL * (sx + sy) + 16384LL * n : 0;
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
        if (lane == 0) s_red[wid] = part;
        if (!half) rp[u] = SDu;            // for the blocks' first deltas
    }
    int it = 1;                            // tabu: the iteration; 2opt: moves made + 1
    if (TABU) ten[t] = blk_tenure(a.seed, (long long)it + t, a.start_id, lo, hi);
    int tpos = 0;
    __syncthreads();
    long long cur = 0;
#pragma unroll
    for (int w = 0; w < TW; ++w) cur += s_red[w];
    cur = ((long long)__builtin_amdgcn_readfirstlane((int)(cur >> 32)) << 32) |
          (unsigned)__builtin_amdgcn_readfirstlane((int)cur);
    long long best = cur;
    const int cap = TABU ? a.iters : (a.iters > 0 ? a.iters : INT32_MAX - 1);

    // the next move, its pair and delta from sel (uniform); false when the search ends here
    int r = 0, s = 0, dstar = 0;
    bool improved = false;
    auto next_move = [&]() -> bool {
        const long long mk = sel[it & 1];
        dstar = __builtin_amdgcn_readfirstlane((int)(mk >> 32));
        const int key = __builtin_amdgcn_readfirstlane((int)mk);
        if (TABU ? dstar == INT32_MAX : dstar >= 0) return false;
        r = key >> 9;
        s = key & 511;
        cur += dstar;
        improved = TABU && cur < best;
        if (improved) best = cur;
        return true;
    };
    // aspiration threshold of the next select: a tabu move is allowed below it
    auto aspire = [&]() -> int {
        const long long d = best - cur;
        return d < -(1 << 24) ? -(1 << 24) : (int)d;
    };
    auto step_tenures = [&]() {
        if (TABU && ++tpos == L) {
            tpos = 0;
            // (read before this by the housekeeping wave in A; written after B2)
            ten[t] = blk_tenure(a.seed, (long long)it + 1 + t, a.start_id, lo, hi);
        }
    };

    if (task) {
        // ================================================================ task waves
        const bool valid = u < n;
        const int duu = D[uc * rs + uc];
        // half 0 of the wave reads D, half 1 reads G
        int8_t *const M = half ? G : D, *const MT = half ? GT : DT;
        const int crow = lane & 15, chunk = (lane >> 4) * 16;   // operand row and 16-byte column
        // operand rows: 16 indices each, blocks 0 and 1 of the wave's 32
        const int row0 = min(wid * 32 + crow, n - 1) * rs + chunk, row1 = min(wid * 32 + 16 + crow, n - 1) * rs + chunk;
        const bool side_s = crow >= 8;     // operand rows 0..7 are side r, 8..15 side s
        while (it <= cap) {
            __syncthreads();   // B1
            if (!next_move()) break;
            const int thr = aspire();
            // ---- A
            const int offr = r * rs, offs = s * rs;
            const int v0 = MT[offr + uc], v1 = MT[offs + uc];                        // x_ur, x_us
            const int v2 = SYM ? v0 : (int)M[offr + uc], v3 = SYM ? v1 : (int)M[offs + uc];   // x_ru, x_su
            const int pk = pack16(v0 - v1, v2 - v3), sums = pack16(v0 + v2, v1 + v3);
            // both halves get both: [0] from D, [1] from G
            const auto pp = __builtin_amdgcn_permlane32_swap(pk, pk, false, false);
            const auto ps = __builtin_amdgcn_permlane32_swap(sums, sums, false, false);
            const int dpk = (int)pp[0], gpk = (int)pp[1], dsm = (int)ps[0], gsm = (int)ps[1];
            const bool apart = u != r && u != s;
            if (half && valid && apart) {
                M[offr + u] = (int8_t)v3;
                M[offs + u] = (int8_t)v2;
                M[u * rs + r] = (int8_t)v1;
                M[u * rs + s] = (int8_t)v0;
                if (!SYM) {
                    MT[offr + u] = (int8_t)v1;
                    MT[offs + u] = (int8_t)v0;
                    MT[u * rs + r] = (int8_t)v3;
                    MT[u * rs + s] = (int8_t)v2;
                }
            }
            // W_u, the index's share of the update in 8-bit limbs.  With x the pair of
            // differences of the wider matrix less 1 (in [-256, 254], two limbs) and y that
            // of the other (in [-127, 127]; minus 1 drops out of every difference), the
            // update of (u, v) is h_u + h_v - x_u.y_v - y_u.x_v, h = x.y = 128 M + L:
            //   half 0  [x limbs | -y twice | L | 1]   half 1  [-M in four limbs | -128 | 0 | 0]
            // and the operand of v is the same with each pair of words exchanged.
            {
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
            }
            SDu -= dot2(dpk, gpk, 0);
            const int dsum = half ? dsm >> 16 : (int)(short)dsm;      // d_ub + d_bu
            const int gsum = half ? (int)(short)gsm : gsm >> 16;      // the same of G under p'
            const int b = half ? s : r;
            __syncthreads();   // B2
            // ---- B: C[b][u] = T'_ub + T'_bu, and SD'_r, SD'_s
            v4i c0 = {0, 0, 0, 0}, c1 = {0, 0, 0, 0}, cs = {0, 0, 0, 0};
            const int so = (side_s ? offs : offr) + chunk;
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int8_t *const Gq = q ? GT : G, *const Dq = q ? DT : D;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    v4i sd = *reinterpret_cast<const v4i *>(Dq + so + 64 * ks);
                    v4i sg = *reinterpret_cast<const v4i *>(Gq + so + 64 * ks);
                    if (ks == KS - 1 && chunk + 64 * ks >= n) {
                        sd = v4i{0, 0, 0, 0};   // past the row: whatever the rows hold there
                        sg = v4i{0, 0, 0, 0};
                    }
                    const v4i g0 = *reinterpret_cast<const v4i *>(Gq + row0 + 64 * ks);
                    const v4i g1 = *reinterpret_cast<const v4i *>(Gq + row1 + 64 * ks);
                    const v4i d0 = *reinterpret_cast<const v4i *>(Dq + row0 + 64 * ks);
                    const v4i d1 = *reinterpret_cast<const v4i *>(Dq + row1 + 64 * ks);
                    c0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(sd, g0, c0, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(sd, g1, c1, 0, 0, 0);
                    cs = __builtin_amdgcn_mfma_i32_16x16x64_i8(sd, sg, cs, 0, 0, 0);
                    c0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(sg, d0, c0, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(sg, d1, c1, 0, 0, 0);
                }
            }
            const int guu = G[uc * rs + uc], dbb = D[b * rs + b], gbb = G[b * rs + b];
            unsigned tb = 0;
            if (TABU) tb = bits[b * NB + wid];
            const int cc = ((lane >> 4) & 1) ? c1[0] : c0[0];
            const int sdr = __builtin_amdgcn_readlane(cs[0], 0), sds = __builtin_amdgcn_readlane(cs[0], 63);
            const int SDr = SYM ? 2 * sdr : sdr, SDs = SYM ? 2 * sds : sds;
            if (u == r) SDu = SDr;
            if (u == s) SDu = SDs;
            int dl = (SYM ? 2 * cc : cc) - SDu - (half ? SDs : SDr) + __mul24(dsum - duu - dbb, gsum - guu - gbb);
            if (!apart) dl = -dstar;       // the move undone
            const bool real = valid && u != b;
            const bool tabu = TABU && ((tb >> l5) & 1u);
            rp[half * NP + u] = !real ? BK_NOMOVE : (tabu ? dl + BK_OFF : dl - BK_OFF);
            const bool adm = real && (!tabu || dl < thr);
            const int d = adm ? dl : INT32_MAX;
            const int wd = wmin32(d);
            if (wd != INT32_MAX) {
                const unsigned long long tie = __ballot(d == wd);
                const int key = (min(u, b) << 9) | max(u, b);
                int wk;
                if (__builtin_popcountll(tie) == 1)
                    wk = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(tie));
                else
                    wk = wmin32(d == wd ? key : KEY_NONE);
                if (lane == 0) sel_min(&sel[(it + 1) & 1], wd, wk);
            }
            step_tenures();
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
        if (TABU) find_events(it + 1, it - 1);
        while (it <= cap) {
            __syncthreads();   // B1
            if (!next_move()) break;
            // ---- A
            if (lane == 0) sel[(it + 1) & 1] = BK_NONE;
            if (lane < 4) {    // the corners of G: (r, r), (r, s), (s, r), (s, s) take (sigma, sigma)
                const int i = lane & 2 ? s : r, j = lane & 1 ? s : r;
                const int si = lane & 2 ? r : s, sj = lane & 1 ? r : s;
                const int8_t x = G[si * rs + sj], y = SYM ? (int8_t)0 : GT[si * rs + sj];
                G[i * rs + j] = x;
                if (!SYM) GT[i * rs + j] = y;
            }
            if (improved)
                for (int x = lane; x < n; x += 64) bestp[x] = perm[x == r ? s : (x == s ? r : x)];
            if (TABU) {
                if (myev >= 0) {
                    const int x = myev >> 9, y = myev & 511;
                    atomicAnd(&bits[x * NB + (y >> 5)], ~(1u << (y & 31)));
                    atomicAnd(&bits[y * NB + (x >> 5)], ~(1u << (x & 31)));
                }
                const int tn = __builtin_amdgcn_readfirstlane(ten[tpos]), pr = (r << 9) | s;
                // still tabu past it + 1 (made by aspiration): its older entry is void
                const unsigned was = __builtin_amdgcn_readfirstlane((int)bits[r * NB + (s >> 5)]);
                if ((was >> (s & 31)) & 1u)
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
            __syncthreads();   // B2
            // ---- B
            if (lane == 0) {
                const int x = perm[r], y = perm[s];
                perm[r] = y;
                perm[s] = x;
            }
            if (TABU) find_events(it + 2, it);
            step_tenures();
            ++it;
        }
    } else {
        // ================================================================ block waves
        const int bw = wid - TW - 1;
        v16i acc[BPW];
        int bI[BPW], bJ[BPW];
        bool has[BPW];
#pragma unroll
        for (int q = 0; q < BPW; ++q) {
            int id = bw * BPW + q;
            has[q] = id < SH::NBLK;
            if (!has[q]) id = SH::NBLK - 1;
            int I = 0;
            while (id >= NB - I) { id -= NB - I; ++I; }
            bI[q] = I;
            bJ[q] = I + id;
        }
        // ---- first deltas: T_ij + T_ji by the contraction, then the rest of Eq. (2)
#pragma unroll
        for (int q = 0; q < BPW; ++q) {
            if (a.table) {   // the caller's neighbourhood of the start
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int x = bI[q] * 32 + 8 * (i >> 2) + 4 * half + (i & 3), v = bJ[q] * 32 + l5;
                    const bool real = x < n && v < n && x != v;
                    acc[q][i] = real ? a.table[pidx(n, min(x, v), max(x, v))] - BK_OFF : BK_NOMOVE;
                }
                continue;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[q][i] = 0;
            const int ri = min(bI[q] * 32 + l5, n - 1) * rs, v = bJ[q] * 32 + l5, vc = min(v, n - 1), rj = vc * rs;
            for (int k = 0; k < n; k += 32) {
                const int kk = k + half * 16;
                const bool in = kk < n;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    const int8_t *const Gq = m ? GT : G, *const Dq = m ? DT : D;
                    v4i gi = *reinterpret_cast<const v4i *>(Gq + ri + kk), di = *reinterpret_cast<const v4i *>(Dq + ri + kk);
                    const v4i gj = *reinterpret_cast<const v4i *>(Gq + rj + kk);
                    const v4i dj = *reinterpret_cast<const v4i *>(Dq + rj + kk);
                    if (!in) gi = di = v4i{0, 0, 0, 0};
                    acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gi, dj, acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(di, gj, acc[q], 0, 0, 0);
                }
            }
            const int dvv = D[rj + vc], gvv = G[rj + vc], sdv = rp[v];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int x = bI[q] * 32 + 8 * (i >> 2) + 4 * half + (i & 3), xc = min(x, n - 1);
                const int dxx = D[xc * rs + xc], gxx = G[xc * rs + xc];
                const int ds = (int)D[xc * rs + vc] + (int)DT[xc * rs + vc] - dxx - dvv;
                const int gs = (int)G[xc * rs + vc] + (int)GT[xc * rs + vc] - gxx - gvv;
                const int full = (SYM ? 2 * acc[q][i] : acc[q][i]) - rp[x] - sdv + __mul24(ds, gs);
                acc[q][i] = x < n && v < n && x != v ? full - BK_OFF : BK_NOMOVE;
            }
        }
        // candidate of the wave's blocks into sel[x]
        auto candidates = [&](int er, int es, int x, int thr) {
            const int thrk = (thr - BK_OFF) * 32;
            int cand = INT32_MAX, cb = 0;
#pragma unroll
            for (int q = 0; q < BPW; ++q) {
                if (BPW > 1 && !has[q]) break;
                int k[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) k[i] = acc[q][i] * 32 + (8 * (i >> 2) + (i & 3));
                int sm_ = min(k[0], k[1]);
                unsigned um = min((unsigned)k[0], (unsigned)k[1]);
#pragma unroll
                for (int i = 2; i < 16; i += 2) {
                    sm_ = min(min(sm_, k[i]), k[i + 1]);
                    if (TABU) um = min(min(um, (unsigned)k[i]), (unsigned)k[i + 1]);
                }
                int c = sm_;
                if (TABU) {
                    const int ta = (int)(um ^ 0x80000000u);   // the lowest tabu slot, as if free
                    c = ta < thrk ? min(sm_, ta) : sm_;
                }
                c |= half << 2;
                const int v = bJ[q] * 32 + l5;
                c = v == er || v == es ? INT32_MAX : c;
                if (q == 0) {
                    cand = c;
                } else {
                    // blocks come in order of I, then J: in one row of blocks the lower row of
                    // a slot decides between equal deltas, across rows the earlier block does
                    const bool take = (c | (bI[q] == bI[q - 1] ? 0 : 31)) < cand;
                    cand = take ? c : cand;
                    cb = take ? q : cb;
                }
            }
            if constexpr (BPW == 1) {
                const int wm = wmin32(cand);
                if (wm < 0) {
                    const int ln = (int)__builtin_ctzll(__ballot(cand == wm));
                    if (lane == 0)
                        sel_min(&sel[x], (wm >> 5) + BK_OFF,
                                ((bI[0] * 32 + (wm & 31)) << 9) | (bJ[0] * 32 + (ln & 31)));
                }
            } else {
                const int d = cand >> 5, wd = wmin32(d);
                if (wd < 0) {
                    int ib = bI[0], jb = bJ[0];
#pragma unroll
                    for (int q = 1; q < BPW; ++q) {
                        ib = cb == q ? bI[q] : ib;
                        jb = cb == q ? bJ[q] : jb;
                    }
                    const int key = ((ib * 32 + (cand & 31)) << 9) | (jb * 32 + l5);
                    const unsigned long long tie = __ballot(d == wd);
                    int wk;
                    if (__builtin_popcountll(tie) == 1)
                        wk = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(tie));
                    else
                        wk = wmin32(d == wd ? key : KEY_NONE);
                    if (lane == 0) sel_min(&sel[x], wd + BK_OFF, wk);
                }
            }
        };
        candidates(-1, -1, it & 1, 0);
        int r0 = -1, s0 = -1;   // the move before: its rows and columns are stale
        while (it <= cap) {
            __syncthreads();   // B1
            if (!next_move()) break;
            const int thr = aspire();
            // ---- A
            if (r0 >= 0) {
#pragma unroll
                for (int q = 0; q < BPW; ++q) {
                    const int I = bI[q], J = bJ[q];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int x = h ? s0 : r0;
                        const int *const src = rp + h * NP;
                        if (I == (x >> 5)) {
                            const int val = src[J * 32 + l5], i = ((x >> 3) & 3) * 4 + (x & 3);
                            const int old = acc[q][i];
                            acc[q][i] = half == ((x >> 2) & 1) ? val : old;
                        }
                        if (J == (x >> 5)) {
                            const bool mine = l5 == (x & 31);
#pragma unroll
                            for (int y = 0; y < 4; ++y) {
                                const v4i val = *reinterpret_cast<const v4i *>(src + I * 32 + 8 * y + 4 * half);
#pragma unroll
                                for (int e = 0; e < 4; ++e) acc[q][4 * y + e] = mine ? val[e] : acc[q][4 * y + e];
                            }
                        }
                    }
                }
            }
            if (TABU) {
                const int cnt = __builtin_amdgcn_readfirstlane(s_ev[0]);
                for (int e = 0; e < cnt; ++e) {
                    const int pr = __builtin_amdgcn_readfirstlane(s_ev[1 + e]);
                    int x = pr >> 9, y = pr & 511;
#pragma unroll
                    for (int m = 0; m < 2; ++m) {   // the slot and, in a diagonal block, its mirror
#pragma unroll
                        for (int q = 0; q < BPW; ++q)
                            if (has[q] && bI[q] == (x >> 5) && bJ[q] == (y >> 5)) {
                                const int i = ((x >> 3) & 3) * 4 + (x & 3);
                                const int old = acc[q][i];
                                acc[q][i] = half == ((x >> 2) & 1) && l5 == (y & 31) ? old - 2 * BK_OFF : old;
                            }
                        const int z = x; x = y; y = z;
                    }
                }
            }
            __syncthreads();   // B2
            // ---- B
#pragma unroll
            for (int q = 0; q < BPW; ++q) {
                if (BPW > 1 && !has[q]) break;
                const v4i wa = Wv[(bI[q] * 32 + l5) * 2 + half], wb = Wv[(bJ[q] * 32 + l5) * 2 + half];
                const v4i wx = {wb[1], wb[0], wb[3], wb[2]};
                acc[q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa, wx, acc[q], 0, 0, 0);
                // rows r and s are the task waves' until the next A
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int x = h ? s : r;
                    if (bI[q] == (x >> 5)) {
                        const int i = ((x >> 3) & 3) * 4 + (x & 3);
                        const int old = acc[q][i];
                        acc[q][i] = half == ((x >> 2) & 1) ? BK_NOMOVE : old;
                    }
                }
            }
            candidates(r, s, (it + 1) & 1, thr);
            r0 = r;
            s0 = s;
            step_tenures();
            ++it;
        }
    }

    // ---- results
    __syncthreads();
    const int *const res = TABU ? bestp : perm;
    for (int x = t; x < n; x += L) a.perm_out[x] = res[x];
    if (t == 0) {
        *a.cost_out = TABU ? best : cur;
        if (a.steps_out) *a.steps_out = it - 1;
    }
}

// Block b runs items[b] of a batch, or search job0 + b of a launch on one instance.
template <int NB, bool SYM, bool TABU>
__global__ void __launch_bounds__(Shape<NB>::LANES) block_kernel(SearchArgs a, BatchArgs b) {
    extern __shared__ __align__(16) unsigned char sm[];
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
    }
    block_body<NB, SYM, TABU>(it, sm);
}

template <int NB, bool SYM, bool TABU>
hipError_t launch_nb(const SearchArgs &a, const BatchArgs &b, int grid, size_t smem, hipStream_t st) {
    hipLaunchKernelGGL((block_kernel<NB, SYM, TABU>), dim3(grid), dim3(Shape<NB>::LANES), smem, st, a, b);
    return report(hipGetLastError(), "block kernel launch");
}

template <bool SYM, bool TABU>
hipError_t launch_any(int nb, const SearchArgs &a, const BatchArgs &b, int grid, size_t smem, hipStream_t st) {
    switch (nb) {
        case 1: return launch_nb<1, SYM, TABU>(a, b, grid, smem, st);
        case 2: return launch_nb<2, SYM, TABU>(a, b, grid, smem, st);
        case 3: return launch_nb<3, SYM, TABU>(a, b, grid, smem, st);
        case 4: return launch_nb<4, SYM, TABU>(a, b, grid, smem, st);
        case 5: return launch_nb<5, SYM, TABU>(a, b, grid, smem, st);
        case 6: return launch_nb<6, SYM, TABU>(a, b, grid, smem, st);
        default: return hipErrorInvalidValue;
    }
}

int blk_lanes(int nb) {
    switch (nb) {
        case 1: return Shape<1>::LANES;
        case 2: return Shape<2>::LANES;
        case 3: return Shape<3>::LANES;
        case 4: return Shape<4>::LANES;
        case 5: return Shape<5>::LANES;
        default: return Shape<6>::LANES;
    }
}

}  // namespace

int block_nb(int n) { return (n + 31) / 32; }

size_t block_smem_bytes(int n, int sym, int hi, bool tabu) {
    const int nb = block_nb(n);
    return (size_t)blk_plan(n, nb, blk_lanes(nb), sym, hi, tabu).total;
}

int block_ok(int n, int sym, int blk, bool tabu, int lo, int hi, size_t max_smem) {
    if (!blk || block_nb(n) > BLOCK_MAX_NB) return 0;
    if (tabu && (hi - lo >= 64 || hi > BLOCK_MAX_TENURE)) return 0;
    return block_smem_bytes(n, sym, hi, tabu) + 1024 <= max_smem ? 1 : 0;   // + its static LDS
}

hipError_t launch_block(bool tabu, int n, int sym, size_t smem, const SearchArgs *a, const BatchArgs *b, int grid,
                        hipStream_t st) {
    if (grid <= 0) return hipSuccess;
    const SearchArgs sa = a ? *a : SearchArgs{};
    const BatchArgs ba = b ? *b : BatchArgs{};
    const int nb = block_nb(n);
    if (tabu)
        return sym ? launch_any<true, true>(nb, sa, ba, grid, smem, st) : launch_any<false, true>(nb, sa, ba, grid, smem, st);
    return sym ? launch_any<true, false>(nb, sa, ba, grid, smem, st) : launch_any<false, false>(nb, sa, ba, grid, smem, st);
}

}  // namespace qapk
