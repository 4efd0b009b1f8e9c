// qap_block_wide.hip -- block form of the tabu and 2opt searches for n = 257 .. 512.
//
// The arithmetic, the slots and the keys are those of the form up to n = 256 (qap_block.h);
// neither F, D nor the whole neighbourhood fit beside a search there, so:
// * eight waves of 256 registers, each with an eighth of the 32 x 32 blocks of Delta: the
//   first 8 (n above 384: 7) in accumulators, then what LDS holds, the others in global
//   scratch, read and written once an iteration;
// * no G = F[p][p]: the rows r and s are recomputed from F and D as they lie in memory, shared
//   by all searches of an instance through L2.  With b = r or s under the new p,
//     T_ub + T_bu = (F x_b + F^T x'_b)[p_u] + (D g_b + D^T g'_b)[u],
//   x_b[p_k] = d_bk, x'_b[p_k] = d_kb, g_b[k] = g_bk, g'_b[k] = g_kb, so the matrices are
//   constant operands of v_mfma_i32_16x16x64_i8, eight of whose rows hold side r, eight side s;
//   their loads run a step of 128 columns ahead of their use, across the barriers, and each
//   block's update and select stand between two steps.
// One iteration (lane t has index u = t in A and C):
//   B1   the minimum is in sel[it & 1]
//   A    W_u, the eight side vectors, SD_u; the ring of moves (one wave)
//   B2
//   B    blocks: the rows and columns of the move before, moves that become free, the update,
//        the candidate for it + 1; the matrix products of rows r and s
//   B3
//   C    the deltas of rows r and s, their candidate; p; the moves that become free next
// There are no tabu bits: the waves whose blocks meet rows r and s leave the signs of their
// slots (32 KB of LDS at n = 512 that hold blocks instead).
// Bound, up to n = 416, by the reads of the matrices from L2 (4 n^2 bytes an iteration and
// search, half for symmetric instances), above also by the scratch blocks (0.4 MB an iteration
// at n = 512, more than L2 holds for 32 searches: 256 searches of 2000 iterations moved 285 GB in
// 55 ms with 64 blocks there, 5.2 TB/s, and move 229 GB in 52 ms with the 51 that are left).
// us per iteration with the tiles streamed through scratch (8 bytes a slot, read and written)
// and here, tables included, 256 searches: n = 300 29.4 and 13.2, n = 512 59.7 and 32.5,
// n = 512 symmetric 50.1 and 26.2; 64 searches n = 400 30.3 and 19.2; one n = 512 39.4 and 23.0.
// Registers decide: with 8 blocks above n = 384, or 16 waves of 128 registers and 4 blocks, the
// kernel spills and takes 43 and 52 us at n = 512.
#include "qap_block.h"

#include <type_traits>

namespace qapk {

namespace {

constexpr int WB_W = 8, WB_L = WB_W * 64;
constexpr int WB_N = 512;                       // indices: one a lane
constexpr int WB_SPAN = 128;                    // tenures: hi - lo below this

// Groups of 16 rows a wave takes in the matrix products (three reach n = 384), and blocks it
// holds in registers: as many as the rest of its 256 leave.
__host__ __device__ constexpr int wb_groups(int n) { return n <= 384 ? 3 : 4; }
__host__ __device__ constexpr int wb_regs(int groups) { return groups == 3 ? 8 : 7; }

// blocks a wave takes
__host__ __device__ inline int wb_per_wave(int n) {
    const int nb = (n + 31) / 32;
    return (nb * (nb + 1) / 2 + WB_W - 1) / WB_W;
}

constexpr int WB_LDS = 160 * 1024 - 2048;   // of the workgroup, beside the kernel's own

struct WbPlan {
    int w, rp, y, vec, perm, fd, ring, blocks, nl, total;   // nl: blocks in LDS
};

__host__ __device__ inline WbPlan wb_plan(int n, int hi, bool tabu) {
    const int nb = (n + 31) / 32, np = nb * 32;
    WbPlan q;
    int o = 0;
    auto take = [&o](int bytes) { int at = o; o += (bytes + 15) & ~15; return at; };
    q.w = take(np * 32);
    q.rp = take(np * 2 * 4);
    q.y = take(np * 4 * 4);      // F's products for r, s, then D's
    q.vec = take(8 * WB_N);
    q.perm = take(np * 4);
    q.fd = take(np * 4);         // f_vv
    q.ring = take(tabu ? blk_ring(hi) * 4 : 0);
    const int fit = (WB_LDS - o) / 4096, rest = WB_W * (wb_per_wave(n) - wb_regs(wb_groups(n)));
    q.nl = rest <= 0 ? 0 : (fit < rest ? fit : rest);
    q.blocks = take(q.nl * 4096);
    q.total = o;
    return q;
}

// f(0), .., f(N - 1), each an instance of its own (registers need constant indices)
template <int N, int Q = 0, class Fn>
__device__ __attribute__((always_inline)) inline void each(Fn &&f) {
    if constexpr (Q < N) {
        f(std::integral_constant<int, Q>{});
        each<N, Q + 1>(f);
    }
}

struct WbShared {
    long long sel[2];
    long long red[WB_W];
    int ev[WB_SPAN + 4];    // the number of pairs that become free, then the pairs
    unsigned tabu[2][WB_N / 32];   // of the pairs of r, and of s, with 32 indices a word
    int tenure;             // of the move
    int bad;
};

template <bool SYM, bool TABU, int WB_G>
__global__ void __launch_bounds__(WB_L) __attribute__((amdgpu_waves_per_eu(2, 2))) wide_block_kernel(SearchArgs a) {
    constexpr int WB_R = wb_regs(WB_G);
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ __align__(16) WbShared sh;
    const int n = a.n, rs = row_stride(n), NB = (n + 31) / 32, NP = NB * 32, KP = (n + 127) / 128;
    const int t = threadIdx.x;
    int lane = t & 63, half = lane >> 5, l5 = lane & 31;
    const int wid = __builtin_amdgcn_readfirstlane(t >> 6);
    const int job = a.job0 + blockIdx.x;
    const int hi = TABU ? a.hi : 0, lo = TABU ? a.lo : 0;
    const WbPlan P = wb_plan(n, hi, TABU);
    const int rmask = blk_ring(hi) - 1;
    v4i *const Wv = reinterpret_cast<v4i *>(sm + P.w);
    int *const rp = reinterpret_cast<int *>(sm + P.rp), *const y = reinterpret_cast<int *>(sm + P.y);
    int8_t *const vec = reinterpret_cast<int8_t *>(sm + P.vec);
    int *const perm = reinterpret_cast<int *>(sm + P.perm), *const fd = reinterpret_cast<int *>(sm + P.fd);
    int *const ring = reinterpret_cast<int *>(sm + P.ring);
    const int32_t *const pin = a.perms_in + (size_t)job * n;
    const int msz = n * rs;                          // bytes of a matrix
    const uint8_t *const F = a.mats, *const FT = F + msz, *const D = F + 2 * msz, *const DT = F + 3 * msz;

    // ---- read and check the start
    int u = t;
    bool valid = u < n;
    const bool active = wid * 64 < n;   // (the other waves have no index)
    if (t == 0) sh.bad = 0;
    for (int i = t; i < NP; i += WB_L) rp[i] = -1;
    for (int i = t; i < NP * 8; i += WB_L) reinterpret_cast<int *>(Wv)[i] = 0;
    for (int i = t; i < 8 * WB_N / 4; i += WB_L) reinterpret_cast<int *>(vec)[i] = 0;
    if (TABU)
        for (int i = t; i <= rmask; i += WB_L) ring[i] = -1;
    if (t < 2) sh.sel[t] = BK_NONE;
    if (t == 0) sh.ev[0] = 0;
    block_sync();
    int pu = valid ? pin[u] : 0;
    if (u < NP) perm[u] = pu;
    if (valid && (pu < 0 || pu >= n || atomicExch(&rp[pu], u) != -1)) sh.bad = 1;
    block_sync();
    if (sh.bad) {
        int32_t *const out = a.perm_out + (size_t)job * n;
        if (out != pin && valid) out[u] = pu;
        if (t == 0) {
            a.cost_out[job] = INT64_MIN;
            if (a.steps_out) a.steps_out[job] = -2;  // QAP_E_NOT_PERM
        }
        return;
    }
    int bp = pu;
    const int dg = valid ? (int)D[u * rs + u] - 128 : 0;   // d_uu
    if (u < NP) fd[u] = valid ? (int)F[u * rs + u] - 128 : 0;

    // ---- SD_i (into rp) and the cost: half a wave takes a row, a lane four columns at a time
    long long part = 0;
    for (int i = t >> 5; i < n; i += WB_L / 32) {
        const int pi = perm[i];
        int sd = 0, raw = 0;
        for (int c = l5 * 4; c < n; c += 128) {
            const unsigned dw = *reinterpret_cast<const unsigned *>(D + i * rs + c);
            const unsigned tw = SYM ? 0 : *reinterpret_cast<const unsigned *>(DT + i * rs + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (c + e >= n) break;
                const int pk = perm[c + e], g = F[pi * rs + pk], d = (dw >> (8 * e)) & 255u;
                raw += g * d;
                sd += (g - 128) * (d - 128);
                if (!SYM) sd += ((int)FT[pi * rs + pk] - 128) * ((int)((tw >> (8 * e)) & 255u) - 128);
            }
        }
        for (int off = 16; off > 0; off >>= 1) {
            sd += __shfl_xor(sd, off, 64);
            raw += __shfl_xor(raw, off, 64);
        }
        if (l5 == 0) rp[i] = SYM ? 2 * sd : sd;
        part += raw;
    }
    part += __shfl_xor(part, 32, 64);
    if (lane == 0) sh.red[wid] = part;
    block_sync();
    long long cur = 0;
#pragma unroll
    for (int w = 0; w < WB_W; ++w) cur += sh.red[w];
    cur = ((long long)__builtin_amdgcn_readfirstlane((int)(cur >> 32)) << 32) |
          (unsigned)__builtin_amdgcn_readfirstlane((int)cur);
    long long best = cur;
    int SDu = valid ? rp[u] : 0;

    // ---- the wave's blocks, in (I, J) order
    const int per = wb_per_wave(n), nblk = NB * (NB + 1) / 2;
    const int first = min(wid * per, nblk), cnt = min(per, nblk - first);
    int I0 = 0, J0 = first;
    while (J0 >= NB - I0 && I0 < NB) {
        J0 -= NB - I0;
        ++I0;
    }
    J0 += I0;
    auto advance = [&](int &I, int &J) __attribute__((always_inline)) {
        if (++J == NB) {
            ++I;
            J = I;
        }
    };
    // the blocks past those in registers: the first of them in LDS, then in scratch
    // (the lower waves take one more where they do not divide)
    const int qmin = P.nl / WB_W, qmore = P.nl % WB_W, ql = qmin + (wid < qmore ? 1 : 0);
    int4 *const near = reinterpret_cast<int4 *>(sm + P.blocks) + (wid * qmin + min(wid, qmore)) * 256;
    int4 *const far = a.tile_work + (size_t)blockIdx.x * a.tile_stride + wid * (per - WB_R - qmin) * 256;
    auto fetch = [&](const int4 *p, v16i &x) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int4 z = p[i * 64 + lane];
            x[4 * i] = z.x, x[4 * i + 1] = z.y, x[4 * i + 2] = z.z, x[4 * i + 3] = z.w;
        }
    };
    auto keep = [&](int4 *p, const v16i &x) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i * 64 + lane] = make_int4(x[4 * i], x[4 * i + 1], x[4 * i + 2], x[4 * i + 3]);
    };
    auto aspire = [&]() -> int {   // a tabu move is allowed below it
        const long long g = best - cur;
        return g < -(1 << 25) ? -(1 << 25) : (int)g;
    };

    // candidate of the wave: c = slot * 32 + row of the block, base its block
    int cand = INT32_MAX, base = 0, pI = -1;
    auto consider = [&](const v16i &acc, int I, int J, int er, int es, int thrk) __attribute__((always_inline)) {
        int k[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) k[i] = acc[i] * 32 + (8 * (i >> 2) + (i & 3));
        int c = min(k[0], k[1]);
        unsigned um = min((unsigned)k[0], (unsigned)k[1]);
#pragma unroll
        for (int i = 2; i < 16; i += 2) {
            c = min(min(c, k[i]), k[i + 1]);
            if (TABU) um = min(min(um, (unsigned)k[i]), (unsigned)k[i + 1]);
        }
        if (TABU) {
            const int ta = (int)(um ^ 0x80000000u);
            c = ta < thrk ? min(c, ta) : c;
        }
        c |= half << 2;
        const int v = J * 32 + l5;
        c = v == er || v == es ? INT32_MAX : c;
        // between equal deltas of one row of blocks the lower row wins, then the earlier block,
        // and across them the earlier row of blocks (whose row bits move to base)
        const int m = I == pI ? 0 : 31;
        base += (cand & m) << 9;
        cand &= ~m;
        const bool take = c < cand;
        cand = take ? c : cand;
        base = take ? (I << 14) | (J << 5) : base;
        pI = I;
    };
    auto publish = [&](int x) __attribute__((always_inline)) {
        const int d = cand >> 5, wd = wmin32(d), key = base + ((cand & 31) << 9) + l5;
        if (wd < 0) {
            const unsigned long long tie = __ballot(d == wd);
            const int wk = __builtin_popcountll(tie) == 1 ? __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(tie))
                                                          : wmin32(d == wd ? key : KEY_NONE);
            if (lane == 0) sel_min(&sh.sel[x & 1], wd + BK_OFF, wk);
        }
        cand = INT32_MAX;
        pI = -1;
    };

    // ---- first neighbourhood, from the table
    v16i acc[WB_R];
    {
        const int32_t *const table = a.table + (size_t)job * a.m;
        const int thrk = (aspire() - BK_OFF) * 32;
        auto read = [&](v16i &x, int I, int J) {
            const int v = J * 32 + l5;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int w = I * 32 + 8 * (i >> 2) + 4 * half + (i & 3);
                x[i] = w < n && v < n && w != v ? table[pidx(n, min(w, v), max(w, v))] - BK_OFF : BK_NOMOVE;
            }
        };
        int I = I0, J = J0;
        each<WB_R>([&](auto q) __attribute__((always_inline)) {
            if (q < cnt) {
                read(acc[q], I, J);
                consider(acc[q], I, J, -1, -1, thrk);
                advance(I, J);
            }
        });
#pragma unroll 1
        for (int q = WB_R; q < cnt; ++q) {
            v16i x;
            read(x, I, J);
            consider(x, I, J, -1, -1, thrk);
            if (q < WB_R + ql)
                keep(near + (q - WB_R) * 256, x);
            else
                keep(far + (q - WB_R - ql) * 256, x);
            advance(I, J);
        }
        publish(1);
    }

    // ---- the products of rows r and s: matrix steps (m, kp) of 128 columns, WB_G groups of 16
    // rows a wave, one step in flight
    constexpr int M = SYM ? 2 : 4;
    int chunk = (lane >> 4) * 16, crow = lane & 15;
    // the last step stays inside the rows (the side vectors are zero past n)
    const int t0 = min(0, rs - 16 - 128 * (KP - 1) - chunk), t1 = min(0, rs - 16 - 128 * (KP - 1) - 64 - chunk);
    unsigned rowo[WB_G];
#pragma unroll
    for (int g = 0; g < WB_G; ++g) rowo[g] = (unsigned)(min((wid + WB_W * g) * 16 + crow, n - 1) * rs + chunk);
    v4i buf[2][WB_G], cc[WB_G];
    int lm = 0, lk = 0, um = 0, uk = 0;   // the next step to load, and to use
    auto load = [&]() __attribute__((always_inline)) {
        const uint8_t *const p = F + (SYM ? 2 * lm : lm) * msz + 128 * lk;
        const bool last = lk == KP - 1;
        const int a0 = last ? t0 : 0, a1 = last ? t1 + 64 : 64;
#pragma unroll
        for (int g = 0; g < WB_G; ++g) {
            buf[0][g] = *reinterpret_cast<const v4i *>(p + (rowo[g] + a0));
            buf[1][g] = *reinterpret_cast<const v4i *>(p + (rowo[g] + a1));
        }
        if (++lk == KP) {
            lk = 0;
            if (++lm == M) lm = 0;
        }
    };
    auto one_step = [&]() __attribute__((always_inline)) {
        if (um == M) return;
        stay_branch();
        const int8_t *const q = vec + (2 * um + (crow >> 3)) * WB_N + chunk + 128 * uk;
        const v4i x0 = *reinterpret_cast<const v4i *>(q), x1 = *reinterpret_cast<const v4i *>(q + 64);
#pragma unroll
        for (int g = 0; g < WB_G; ++g) {
            cc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, buf[0][g] ^ (int)0x80808080, cc[g], 0, 0, 0);
            cc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, buf[1][g] ^ (int)0x80808080, cc[g], 0, 0, 0);
        }
        load();
        if (++uk == KP) {
            uk = 0;
            ++um;
            if (SYM || um == 2 || um == 4) {   // F's or D's products are whole
                stay_branch();
                int *const o = y + ((um == M ? 2 : 0) + half) * NP;
                if (!(lane & 16))
#pragma unroll
                    for (int g = 0; g < WB_G; ++g) {
                        const int v = (wid + WB_W * g) * 16 + crow;
                        if (v < NP) o[v] = cc[g][0];
                    }
#pragma unroll
                for (int g = 0; g < WB_G; ++g) cc[g] = v4i{0, 0, 0, 0};
            }
        }
    };
#pragma unroll
    for (int g = 0; g < WB_G; ++g) cc[g] = v4i{0, 0, 0, 0};
    load();

    // ---- the wave that keeps the tabu list
    const bool keeper = TABU && wid == WB_W - 1;
    // pairs whose latest tenure ends at iteration x, among moves up to `last`
    auto find_events = [&](int x, int last) {
        int c = 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int tn = lo + lane + 64 * j, i = x - tn;
            int ev = -1;
            if (tn <= hi && i <= last) {
                const int e = ring[i & rmask];
                if ((e >> 18) == tn) ev = e & 0x3ffff;
            }
            const unsigned long long m = __ballot(ev >= 0);
            if (ev >= 0) sh.ev[1 + c + __builtin_popcountll(m & ((1ull << lane) - 1))] = ev;
            c += __builtin_popcountll(m);
        }
        if (lane == 0) sh.ev[0] = c;
    };
    int tens = 0;   // of iterations it0 + lane, it0 = 1, 65, ..
    auto draw = [&](int it0) {
        Tenures x;
        x.begin(a.seed, (long long)it0 + lane, a.start_base + job);
#pragma unroll 1
        for (int i = 0; i < 10; ++i) x.round();
        tens = x.value(lo, hi);
    };
    if (keeper) {
        draw(1);
        find_events(2, 0);
    }

    const int cap = TABU ? a.iters : (a.iters > 0 ? a.iters : INT32_MAX - 1);
    int it = 1, r0 = 1 << 14, s0 = 1 << 14;   // the move before (none)
    while (it <= cap) {
        // (addresses of the lane's index are made where they are used, not kept throughout)
        asm volatile("" : "+v"(lane));
        half = lane >> 5, l5 = lane & 31, chunk = (lane >> 4) * 16, crow = lane & 15;
        u = wid * 64 + lane;
        valid = u < n;
        block_sync();   // B1
        const long long mk = sh.sel[it & 1];
        const int dstar = __builtin_amdgcn_readfirstlane((int)(mk >> 32));
        const int key = __builtin_amdgcn_readfirstlane((int)mk);
        if (TABU ? dstar == INT32_MAX : dstar >= 0) break;
        const int r = key >> 9, s = key & 511;
        cur += dstar;
        const bool improved = TABU && cur < best;
        if (improved) best = cur;
        const int thr = aspire();
        // ---- A
        const int pr = __builtin_amdgcn_readfirstlane(perm[r]), ps = __builtin_amdgcn_readfirstlane(perm[s]);
        if (u == 0) sh.sel[(it + 1) & 1] = BK_NONE;
        pu = u == r ? ps : (u == s ? pr : pu);
        if (improved) bp = pu;
        if (keeper) {
            const int pair = (r << 9) | s, tn = __builtin_amdgcn_readlane(tens, (it - 1) & 63);
            // only a new best may be tabu (aspiration): the pair's older entry is void
            if (improved)
                for (int x = lane; x <= rmask; x += 64) {
                    const int e = ring[x];
                    if (e >= 0 && (e & 0x3ffff) == pair) ring[x] = -1;
                }
            if (lane == 0) {
                ring[it & rmask] = (tn << 18) | pair;
                sh.tenure = tn;
            }
        }
        int dsum = 0, gsum = 0;
        if (active) {
            const int uc = min(u, n - 1);
            // d_ur, d_us, d_ru, d_su, and the same of G under the new p
            const int d2 = (int)D[r * rs + uc] - 128, d3 = (int)D[s * rs + uc] - 128;
            const int g2 = (int)F[ps * rs + pu] - 128, g3 = (int)F[pr * rs + pu] - 128;
            const int d0 = SYM ? d2 : (int)DT[r * rs + uc] - 128, d1 = SYM ? d3 : (int)DT[s * rs + uc] - 128;
            const int g0 = SYM ? g2 : (int)FT[ps * rs + pu] - 128, g1 = SYM ? g3 : (int)FT[pr * rs + pu] - 128;
            const int dbr = (int)D[r * rs + r] - 128, dbs = (int)D[s * rs + s] - 128;
            // (before the move g_ur was what g_us is now, for u other than r and s)
            const int dpk = pack16(d0 - d1, d2 - d3), gpk = pack16(g1 - g0, g3 - g2);
            // d_ub + d_bu - d_uu - d_bb and g_ub + g_bu, for b = r and s
            dsum = pack16(d0 + d2 - dg - dbr, d1 + d3 - dg - dbs);
            gsum = pack16(g0 + g2, g1 + g3);
            SDu -= dot2(dpk, gpk, 0);
            {   // W_u, as up to n = 256: both halves
                const int xp = a.blk == 1 ? dpk : gpk, yp = a.blk == 1 ? gpk : dpk;
                const int x = pk_add(xp, -1), xa = pk_ashr<1>(x), xb = pk_sub(x, xa);
                const int X = bperm((unsigned)xb, (unsigned)xa, 0x06020400u);
                const int yn = pk_sub(0, yp), Y = bperm((unsigned)yn, (unsigned)yn, 0x02020000u);
                const int h = dot2(x, yp, 0), Mh = (h + 64) >> 7, Lh = h - (Mh << 7);
                const int mm = pack16(-Mh, -Mh);
                const int m01 = pk_ashr<2>(pk_add(mm, 0x00010000)), m23 = pk_ashr<2>(pk_add(mm, 0x00030002));
                const int H = bperm((unsigned)m23, (unsigned)m01, 0x06040200u);
                if (valid) {
                    Wv[u * 2] = v4i{X, Y, Lh & 0xff, 1};
                    Wv[u * 2 + 1] = v4i{H, (int)0x80808080, 0, 0};
                    vec[pu] = (int8_t)d2;
                    vec[WB_N + pu] = (int8_t)d3;
                    if (!SYM) {
                        vec[2 * WB_N + pu] = (int8_t)d0;
                        vec[3 * WB_N + pu] = (int8_t)d1;
                    }
                    int8_t *const gv = vec + (SYM ? 2 : 4) * WB_N;
                    gv[u] = (int8_t)g2;
                    gv[WB_N + u] = (int8_t)g3;
                    if (!SYM) {
                        gv[2 * WB_N + u] = (int8_t)g0;
                        gv[3 * WB_N + u] = (int8_t)g1;
                    }
                }
            }
        }
        block_sync();   // B2
        // ---- B
        um = uk = 0;
        const int thrk = (thr - BK_OFF) * 32;
        const int nev = TABU ? __builtin_amdgcn_readfirstlane(sh.ev[0]) : 0;
        const int ev0 = TABU ? __builtin_amdgcn_readfirstlane(sh.ev[1]) : 0;
        auto set_row = [&](v16i &x, int w, int val) __attribute__((always_inline)) {
            const int i = ((w >> 3) & 3) * 4 + (w & 3), old = x[i];
            x[i] = half == ((w >> 2) & 1) ? val : old;
        };
        // rows and columns of blocks that have more to do than the update
        unsigned hitI = (1u << (r >> 5)) | (1u << (s >> 5));
        if (it > 1) hitI |= (1u << (r0 >> 5)) | (1u << (s0 >> 5));
        const unsigned hitJ = hitI;
        if (TABU)
            for (int e = 0; e < nev; ++e) hitI |= 1u << ((e == 0 ? ev0 : __builtin_amdgcn_readfirstlane(sh.ev[1 + e])) >> 14);
        auto repair = [&](v16i &x, int I, int J) __attribute__((always_inline)) {
            // the rows and columns of the move before take the deltas recomputed for them
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int w = h ? s0 : r0;
                if (I == w >> 5) {
                    stay_branch();
                    set_row(x, w, rp[h * NP + J * 32 + l5]);
                }
                if (J == w >> 5) {
                    stay_branch();
                    const bool mine = l5 == (w & 31);
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const v4i val = *reinterpret_cast<const v4i *>(rp + h * NP + I * 32 + 8 * z + 4 * half);
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[4 * z + e] = mine ? val[e] : x[4 * z + e];
                    }
                }
            }
            if (TABU)   // moves that are free from it + 1 on
                for (int e = 0; e < nev; ++e) {
                    const int pair = e == 0 ? ev0 : __builtin_amdgcn_readfirstlane(sh.ev[1 + e]);
                    const int w = pair >> 9, z = pair & 511;
                    if ((w >> 5) != I || (z >> 5) != J) continue;
                    stay_branch();
                    const int i = ((w >> 3) & 3) * 4 + (w & 3), old = x[i];
                    x[i] = half == ((w >> 2) & 1) && l5 == (z & 31) ? old - 2 * BK_OFF : old;
                    if (I == J) {   // the mirror slot of a diagonal block
                        stay_branch();
                        const int j = ((z >> 3) & 3) * 4 + (z & 3), ol2 = x[j];
                        x[j] = half == ((z >> 2) & 1) && l5 == (w & 31) ? ol2 - 2 * BK_OFF : ol2;
                    }
                }
            // rows and columns r and s: the tabu state of their slots, for C; rows: out of the
            // minimum until they are recomputed
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int w = h ? s : r;
                if (TABU && J == w >> 5 && I != J) {
                    stay_branch();
                    unsigned free = 0;   // of the half's rows of the column
#pragma unroll
                    for (int i = 0; i < 16; ++i) free |= ((unsigned)x[i] >> 31) << (8 * (i >> 2) + (i & 3));
                    free = half ? free << 4 : free;
                    const unsigned both = (unsigned)__builtin_amdgcn_readlane((int)free, w & 31) |
                                          (unsigned)__builtin_amdgcn_readlane((int)free, 32 + (w & 31));
                    if (lane == 0) sh.tabu[h][I] = ~both;
                }
                if (I != w >> 5) continue;
                stay_branch();
                const int i = ((w >> 3) & 3) * 4 + (w & 3), old = x[i];
                if (TABU) {
                    const unsigned long long m = __ballot(old > 0);
                    if (lane == 0) sh.tabu[h][J] = (unsigned)(((w >> 2) & 1) ? m >> 32 : m);
                }
                x[i] = half == ((w >> 2) & 1) ? BK_NOMOVE - (1 << 20) : old;
            }
        };
        auto process = [&](v16i &x, int I, int J) __attribute__((always_inline)) {
            if (((hitI >> I) | (hitJ >> J)) & 1) {
                stay_branch();
                repair(x, I, J);
            }
            const v4i wa = Wv[(I * 32 + l5) * 2 + half], wb = Wv[(J * 32 + l5) * 2 + half];
            const v4i wx = {wb[1], wb[0], wb[3], wb[2]};
            x = __builtin_amdgcn_mfma_i32_32x32x32_i8(wa, wx, x, 0, 0, 0);
            consider(x, I, J, r, s, thrk);
        };
        {
            int I = I0, J = J0;
            // (what a block needs is made when its turn comes, not kept for all of them)
            int ij = I << 8 | J;
            asm volatile("" : "+v"(ij));
            ij = __builtin_amdgcn_readfirstlane(ij);
            I = ij >> 8;
            J = ij & 255;
            each<WB_R>([&](auto q) __attribute__((always_inline)) {
                if (q < cnt) {
                    process(acc[q], I, J);
                    one_step();
                    advance(I, J);
                }
            });
            const int inl = min(ql, cnt - WB_R), inw = cnt - WB_R - ql;
#pragma unroll 1
            for (int q = 0; q < inl; ++q) {
                v16i x;
                fetch(near + q * 256, x);
                process(x, I, J);
                keep(near + q * 256, x);
                one_step();
                advance(I, J);
            }
#pragma unroll 1
            for (int q = 0; q < inw; ++q) {
                v16i x;
                fetch(far + q * 256, x);
                one_step();
                process(x, I, J);
                keep(far + q * 256, x);
                advance(I, J);
            }
#pragma unroll 1
            while (um != M) one_step();
        }
        publish(it + 1);
        block_sync();   // B3
        // ---- C
        if (active) {
            const int uy = min(u, NP - 1);
            const int cr = y[pu] + y[2 * NP + uy], cs = y[NP + pu] + y[3 * NP + uy];
            const int qr = y[ps] + y[2 * NP + r], qs = y[NP + pr] + y[3 * NP + s];   // T_rr, T_ss twice
            const int SDr = SYM ? qr : qr / 2, SDs = SYM ? qs : qs / 2;
            const int fu = fd[pu], fr = fd[ps], fs = fd[pr];
            if (u == r) SDu = SDr;
            if (u == s) SDu = SDs;
            int dr = (SYM ? 2 * cr : cr) - SDu - SDr + __mul24((int)(short)dsum, (int)(short)gsum - fu - fr);
            int ds = (SYM ? 2 * cs : cs) - SDu - SDs + __mul24(dsum >> 16, (gsum >> 16) - fu - fs);
            if (u == s) dr = -dstar;   // the move undone
            if (u == r) ds = -dstar;
            const bool realr = valid && u != r, reals = valid && u != s;
            bool tr = false, ts = false;
            if (TABU) {
                const bool made = sh.tenure >= 2;   // the move itself is tabu at it + 1
                const unsigned wr = sh.tabu[0][uy >> 5], ws = sh.tabu[1][uy >> 5];
                tr = realr && (u == s ? made : (wr >> (u & 31)) & 1u);
                ts = reals && (u == r ? made : (ws >> (u & 31)) & 1u);
            }
            if (u < NP) {
                rp[u] = !realr ? BK_NOMOVE : (tr ? dr + BK_OFF : dr - BK_OFF);
                rp[NP + u] = !reals ? BK_NOMOVE : (ts ? ds + BK_OFF : ds - BK_OFF);
            }
            int d = realr && (!tr || dr < thr) ? dr : INT32_MAX, k = (min(u, r) << 9) | max(u, r);
            const int e = reals && (!ts || ds < thr) ? ds : INT32_MAX, ke = (min(u, s) << 9) | max(u, s);
            const bool take = e < d || (e == d && ke < k);
            d = take ? e : d;
            k = take ? ke : k;
            const int wd = wmin32(d);
            if (wd != INT32_MAX) {
                const unsigned long long tie = __ballot(d == wd);
                const int wk = __builtin_popcountll(tie) == 1 ? __builtin_amdgcn_readlane(k, (int)__builtin_ctzll(tie))
                                                              : wmin32(d == wd ? k : KEY_NONE);
                if (lane == 0) sel_min(&sh.sel[(it + 1) & 1], wd, wk);
            }
            if (u == r || u == s) perm[u] = pu;
        }
        if (keeper) {
            find_events(it + 2, it);
            if ((it & 63) == 0) draw(it + 1);
        }
        r0 = r;
        s0 = s;
        ++it;
    }

    // ---- results
    if (valid) a.perm_out[(size_t)job * n + u] = TABU ? bp : pu;
    if (t == 0) {
        a.cost_out[job] = TABU ? best : cur;
        if (a.steps_out) a.steps_out[job] = it - 1;
    }
}

}  // namespace

// Whether a launch of tabu or 2opt searches above n = 256 runs in block form.
int wide_block_ok(bool tabu, const SearchArgs &a, size_t max_smem) {
    if (!a.blk || a.freq || a.n <= WIDE_N || a.n > WB_N) return 0;
    if (tabu && (a.hi - a.lo >= WB_SPAN || a.hi > BLOCK_MAX_TENURE)) return 0;
    const WbPlan p = wb_plan(a.n, tabu ? a.hi : 0, tabu);
    const int spill = wb_per_wave(a.n) - wb_regs(wb_groups(a.n)) - p.nl / WB_W;   // blocks of a wave in scratch
    if (spill > 0 && (long long)spill * WB_W * 256 > a.tile_stride) return 0;
    return (size_t)p.total + 2048 <= max_smem ? 1 : 0;
}

hipError_t launch_wide_block(bool tabu, const SearchArgs &a, int grid, hipStream_t st) {
    const size_t smem = (size_t)wb_plan(a.n, tabu ? a.hi : 0, tabu).total;
    const dim3 g(grid), b(WB_L);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, smem, st, a); };
    auto form = [&](auto sym, auto tab) {
        wb_groups(a.n) == 3 ? go(wide_block_kernel<sym, tab, 3>) : go(wide_block_kernel<sym, tab, 4>);
    };
    if (tabu)
        a.sym ? form(std::true_type{}, std::true_type{}) : form(std::false_type{}, std::true_type{});
    else
        a.sym ? form(std::true_type{}, std::false_type{}) : form(std::false_type{}, std::false_type{});
    return report(hipGetLastError(), "wide block kernel launch");
}

}  // namespace qapk
