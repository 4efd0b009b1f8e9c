// qap_table.hip -- cost (Eq. 1) and whole-neighbourhood (Eq. 2) kernels.
//
// One workgroup per start; every entry of F and D lies in [0, 255].
#include "qap_internal.h"

namespace qapk {

namespace {

__device__ inline long long wave_sum64(long long v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// costs[j] = sum_i sum_k F[p_i][p_k] D[i][k]   (Eq. 1)
//
// The lane's share of Eq. (1) of one start, 256 lanes: half a wave takes a row, a lane four
// columns at a time, so that a lane's columns of p stay in registers and its work is four byte
// gathers a word of D, which is read from global memory in order.  (One lane a row, its
// columns one after the other, left 155 of 256 lanes idle at n = 101 and made 101 steps of
// three reads instead of 13 of five.)  us a call, before and now, where a call's host work is
// 7.9: 1024 starts n = 101 8.8 and 7.9, n = 128 11.1 and 8.1, 256 starts n = 256 12.1 and 9.0,
// n = 512 177 and 43.
__device__ __attribute__((always_inline)) inline int cost_part(int n, int rs, const uint8_t *F, const uint8_t *D,
                                                               const int *perm) {
    const int t = threadIdx.x;
    int acc = 0;   // at most 64 rows of 16 entries below 2^16
    for (int c = (t & 31) * 4; c < n; c += 128) {
        int pc[4];
        unsigned in = 0;   // the columns below n
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            pc[e] = c + e < n ? perm[c + e] : 0;
            if (c + e < n) in |= 0xffu << (8 * e);
        }
#pragma unroll 4
        for (int i = t >> 5; i < n; i += 8) {
            const unsigned d = *reinterpret_cast<const unsigned *>(D + i * rs + c) & in;
            const uint8_t *const f = F + perm[i] * rs;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc += (int)f[pc[e]] * (int)((d >> (8 * e)) & 255u);
        }
    }
    return acc;
}

// The start and F (bytes) in LDS.  Bound by latency: the launch, the staging and the gathers.
__global__ void __launch_bounds__(256) cost_kernel(TableArgs a) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int bad;
    __shared__ long long red[4];
    const int n = a.n, rs = row_stride(n), job = blockIdx.x, t = threadIdx.x;
    uint8_t *Fm = sm;
    int *perm = reinterpret_cast<int *>(sm + n * rs);
    int *pinv = perm + n;
    const int32_t *const p = a.perms + (size_t)job * n;
    const int mine = t < n ? p[t] : 0;   // n <= 256
    const uint4 *src = reinterpret_cast<const uint4 *>(a.mats);
    for (int i = t; i < n * rs / 16; i += 256) reinterpret_cast<uint4 *>(Fm)[i] = src[i];
    if (t == 0) bad = 0;
    if (t < n) {
        pinv[t] = -1;
        perm[t] = mine;
    }
    __syncthreads();
    if (t < n && (mine < 0 || mine >= n || atomicExch(&pinv[mine], t) != -1)) bad = 1;
    __syncthreads();
    if (bad) {
        if (t == 0) a.costs[job] = INT64_MIN;
        return;
    }
    long long part = cost_part(n, rs, Fm, a.mats + (size_t)2 * n * rs, perm);
    part = wave_sum64(part);
    if ((t & 63) == 0) red[t >> 6] = part;
    __syncthreads();
    if (t == 0) {
        long long z = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) z += red[w];
        a.costs[job] = z;
    }
}

// ---- whole neighbourhood (a3) as integer contractions on the matrix cores
//
// With G = F[p][p] (G[a][b] = F[p_a][p_b]) and T = G.D^T + G^T.D, every delta of Eq. (2)
// (with its diagonal term) is
//   delta(i, j) = T_ij + T_ji - T_ii - T_jj + (d_ij + d_ji - d_ii - d_jj)(g_ij + g_ji - g_ii - g_jj)
// (expanding Eq. (2) and collecting the k = i, j terms, which factor).  No delta changes when
// a constant is added to every entry of F or of D, so the contractions run as
// v_mfma_i32_32x32x32_i8 on entries minus 128 and nothing is corrected.
// A workgroup takes one start: X = G, Y = D in LDS (int8, zero past n); a wave takes pairs of
// 32 x 32 output tiles (I <= J) and accumulates T_ij + T_ji as X_I.Y_J^T + Y_I.X_J^T over the
// rows and, unless F and D are both symmetric, the same over the columns, which the transposing
// LDS reads give without a transposed copy.
// Bound by the gathers and reads of LDS beside the table's own bytes.  1024 starts, us, before
// (transposed matrices staged in a second phase, the shift undone from row sums, the k = i, j
// terms from eight byte reads an entry) and now: n = 64 (256 starts) 12.8 and 7.9, 101 59.6 and 27.2, 128
// symmetric 45.9 and 28.4 (33 MB written), 128 66.3 and 32.2, 200 61.5 and 31.3 (256 starts),
// 256 84.2 and 43.7 (256 starts).

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int TB_LANES = 512, TB_W = TB_LANES / 64;

__host__ __device__ inline int tb_rows(int n) { return (n + 31) & ~31; }
// LDS rows: an odd multiple of 16 bytes
__host__ __device__ inline int tb_stride(int n) { return (((n + 15) / 16) | 1) * 16; }

struct TbPlan {
    int perm, pinv, sd, dg, x, y, total;
};

__host__ __device__ inline TbPlan tb_plan(int n) {
    const int rs = tb_stride(n), np = tb_rows(n);
    TbPlan q;
    int o = 0;
    q.perm = o; o += np * 4;
    q.pinv = o; o += np * 4;
    q.sd = o;   o += np * 4;   // T_ii
    q.dg = o;   o += np * 4;   // d_ii | g_ii << 16
    q.x = o;    o += ((n + 15) & ~15) * rs;
    q.y = o;    o += ((n + 15) & ~15) * rs;
    o += 64;                   // the last row's reads past n
    q.total = o;
    return q;
}

// Read and check one start into LDS (perm and its inverse); false if it is not a
// permutation of 0..n-1.  Ends with a barrier.
__device__ bool tb_stage_perm(const int32_t *p, int n, int *perm, int *pinv, int *bad) {
    const int L = blockDim.x, t = threadIdx.x;
    if (t == 0) *bad = 0;
    for (int u = t; u < n; u += L) pinv[u] = -1;
    __syncthreads();
    for (int u = t; u < n; u += L) {
        const int v = p[u];
        perm[u] = v;
        if (v < 0 || v >= n || atomicExch(&pinv[v], u) != -1) *bad = 1;
    }
    __syncthreads();
    return *bad == 0;
}

// n above WIDE_N (F and D do not fit in LDS): the matrices are read in place from global
// memory, only the start and its inverse are staged.

// Cost (Eq. 1) of one start per workgroup.
__global__ void __launch_bounds__(256) cost_wide_kernel(TableArgs a) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int bad;
    __shared__ long long red[4];
    const int n = a.n, rs = row_stride(n), job = blockIdx.x, t = threadIdx.x;
    int *perm = reinterpret_cast<int *>(sm), *pinv = perm + n;
    if (!tb_stage_perm(a.perms + (size_t)job * n, n, perm, pinv, &bad)) {
        if (t == 0) a.costs[job] = INT64_MIN;
        return;
    }
    long long part = cost_part(n, rs, a.mats, a.mats + (size_t)2 * n * rs, perm);
    part = wave_sum64(part);
    if ((t & 63) == 0) red[t >> 6] = part;
    __syncthreads();
    if (t == 0) {
        long long z = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) z += red[w];
        a.costs[job] = z;
    }
}

// (I, J), I <= J, of pair q in row-major order over nt x nt
__device__ inline void tb_pair(int q, int nt, int &I, int &J) {
    I = 0;
    while (q >= nt - I) {
        q -= nt - I;
        ++I;
    }
    J = I + q;
}

__device__ inline long long tb_load8(const uint8_t *p) { return *reinterpret_cast<const long long *>(p); }

// ---- whole neighbourhood above WIDE_N: the same contraction, blocked
//
// X = G' and Y = D' no longer fit in LDS for a whole start, so a workgroup takes one pair
// (BI <= BJ) of 128-row blocks of one start and streams k through LDS in chunks of
// TW_KC: each chunk stages X and Y of both row blocks (X gathered from global F through
// the permutation, Y read from global D, both shifted to int8), adds its part of the row
// sums and diagonal terms of those rows, and accumulates the 32 x 32 output tiles of the
// pair (two per wave) with v_mfma_i32_32x32x16_i8.  The epilogue undoes the
// shift from the row sums and adds the k = i, j terms one by one, with the entries of D and G
// at (i, j), (j, i), (i, i), (j, j) read from global memory.  Bound by the gathers of X: four go out at once, without a branch,
// beside one word of Y (entry by entry, each behind its test, 256 starts at n = 512 took 860
// us, symmetric 516, 64 at n = 300 122; now 622, 402 and 87).

constexpr int TW_ROWS = 128;                 // rows of a block
constexpr int TW_KC = 128;                   // k per chunk
constexpr int TW_RS = TW_KC + 16;            // LDS row stride of a staged chunk
constexpr int TW_TILES = TW_ROWS / 32;       // 32 x 32 tiles per block side

struct TwPlan {
    int perm, xi, yi, xj, yj, ui, uj, ti, tj, total;
};

__host__ __device__ inline TwPlan tw_plan(int n) {
    TwPlan q;
    int o = 0;
    q.perm = o; o += ((n + 3) & ~3) * 4;
    o = (o + 255) & ~255;
    q.xi = o; o += TW_ROWS * TW_RS;
    q.yi = o; o += TW_ROWS * TW_RS;
    q.xj = o; o += TW_ROWS * TW_RS;
    q.yj = o; o += TW_ROWS * TW_RS;
    q.ui = o; o += TW_ROWS * 4;
    q.uj = o; o += TW_ROWS * 4;
    q.ti = o; o += TW_ROWS * 4;
    q.tj = o; o += TW_ROWS * 4;
    q.total = o;
    return q;
}

__global__ void __launch_bounds__(TB_LANES) table_wide_mfma_kernel(TableArgs a) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int bad;
    const int n = a.n, rs = row_stride(n), job = blockIdx.y, t = threadIdx.x, L = blockDim.x;
    const int lane = t & 63, w = t >> 6;
    const TwPlan P = tw_plan(n);
    int32_t *out = a.table + (size_t)job * a.m;
    int *perm = reinterpret_cast<int *>(sm + P.perm);
    int *U_i = reinterpret_cast<int *>(sm + P.ui), *U_j = reinterpret_cast<int *>(sm + P.uj);
    int *T_i = reinterpret_cast<int *>(sm + P.ti), *T_j = reinterpret_cast<int *>(sm + P.tj);
    uint8_t *Xi = sm + P.xi, *Yi = sm + P.yi, *Xj = sm + P.xj, *Yj = sm + P.yj;
    const int nb = (n + TW_ROWS - 1) / TW_ROWS;
    int BI, BJ;
    tb_pair(blockIdx.x, nb, BI, BJ);
    const bool same = BI == BJ;
    // check the start (its inverse in the X chunk buffer, which is free until staging)
    {
        int *pinv = reinterpret_cast<int *>(Xi);
        if (t == 0) bad = 0;
        for (int u = t; u < n; u += L) pinv[u] = -1;
        __syncthreads();
        const int32_t *p = a.perms + (size_t)job * n;
        for (int u = t; u < n; u += L) {
            const int v = p[u];
            perm[u] = v;
            if (v < 0 || v >= n || atomicExch(&pinv[v], u) != -1) bad = 1;
        }
        __syncthreads();
        if (bad) {
            // every block of the start clears its own entries
            for (int x = t; x < TW_ROWS * TW_ROWS; x += L) {
                const int i = BI * TW_ROWS + x / TW_ROWS, j = BJ * TW_ROWS + x % TW_ROWS;
                if (i < j && j < n) out[pidx(n, i, j)] = 0;
            }
            return;
        }
    }
    for (int x = t; x < TW_ROWS; x += L) U_i[x] = U_j[x] = T_i[x] = T_j[x] = 0;

    // the wave's output tiles: (ti, tj) in the pair, ti <= tj when the blocks are the same
    const int ntiles = same ? TW_TILES * (TW_TILES + 1) / 2 : TW_TILES * TW_TILES;
    int tI[2], tJ[2];
    bool has[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int id = w + 8 * q;
        has[q] = id < ntiles;
        if (same) {
            tb_pair(has[q] ? id : 0, TW_TILES, tI[q], tJ[q]);
        } else {
            tI[q] = id / TW_TILES;
            tJ[q] = id % TW_TILES;
        }
    }
    v16i acc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[q][r] = 0;

    // per row of the two blocks (threads 0 .. 2 TW_ROWS - 1): sum x', sum y', sum x y
    int sx = 0, sy = 0, dxy = 0, u_acc = 0, t_acc = 0;
    const int phases = a.sym ? 1 : 2;
    const int wpr = TW_KC / 4;   // words per staged row
    for (int ph = 0; ph < phases; ++ph) {
        const uint8_t *Fp = a.mats + (size_t)(ph ? 1 : 0) * n * rs;   // F, then F^T
        const uint8_t *Dp = a.mats + (size_t)(ph ? 3 : 2) * n * rs;   // D, then D^T
        sx = sy = dxy = 0;
        for (int k0 = 0; k0 < n; k0 += TW_KC) {
            __syncthreads();   // the previous chunk is consumed
            const int sides = same ? 1 : 2;
            for (int v = t; v < sides * TW_ROWS * wpr; v += L) {
                const int side = v / (TW_ROWS * wpr), rem = v - side * TW_ROWS * wpr;
                const int ri = rem / wpr, c = (rem - ri * wpr) * 4;
                const int i = (side ? BJ : BI) * TW_ROWS + ri, k = k0 + c;
                unsigned xw = 0, yw = 0;
                if (i < n && k < n) {
                    // (four gathers at once, masked past n, where rows and perm are padded)
                    const uint8_t *frow = Fp + (size_t)perm[i] * rs;
                    const int4 pk = *reinterpret_cast<const int4 *>(perm + k);
                    const int real = n - k;
                    const unsigned in = real >= 4 ? ~0u : 0xffffffffu >> (8 * (4 - real));
                    const unsigned f0 = frow[pk.x], f1 = frow[real > 1 ? pk.y : 0], f2 = frow[real > 2 ? pk.z : 0],
                                   f3 = frow[real > 3 ? pk.w : 0];
                    xw = ((f0 | f1 << 8 | f2 << 16 | f3 << 24) ^ 0x80808080u) & in;
                    yw = (*reinterpret_cast<const unsigned *>(Dp + (size_t)i * rs + k) ^ 0x80808080u) & in;
                }
                reinterpret_cast<unsigned *>(side ? Xj : Xi)[(ri * TW_RS + c) / 4] = xw;
                reinterpret_cast<unsigned *>(side ? Yj : Yi)[(ri * TW_RS + c) / 4] = yw;
            }
            __syncthreads();
            // row sums and diagonal terms of this chunk
            if (t < (same ? 1 : 2) * TW_ROWS) {
                const int side = t / TW_ROWS, ri = t - side * TW_ROWS;
                const int *xr = reinterpret_cast<const int *>((side ? Xj : Xi) + ri * TW_RS);
                const int *yr = reinterpret_cast<const int *>((side ? Yj : Yi) + ri * TW_RS);
                for (int c = 0; c < wpr; ++c) {
                    sx = __builtin_amdgcn_sdot4(xr[c], 0x01010101, sx, false);
                    sy = __builtin_amdgcn_sdot4(yr[c], 0x01010101, sy, false);
                    dxy = __builtin_amdgcn_sdot4(xr[c], yr[c], dxy, false);
                }
            }
            // S += X_I . Y_J^T + Y_I . X_J^T over this chunk
            const int row = lane & 31, kh = 8 * (lane >> 5);
            const uint8_t *XJ = same ? Xi : Xj, *YJ = same ? Yi : Yj;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (!has[q]) continue;
                const uint8_t *xi = Xi + (tI[q] * 32 + row) * TW_RS + kh, *yj = YJ + (tJ[q] * 32 + row) * TW_RS + kh;
                const uint8_t *yi = Yi + (tI[q] * 32 + row) * TW_RS + kh, *xj = XJ + (tJ[q] * 32 + row) * TW_RS + kh;
#pragma unroll
                for (int kk = 0; kk < TW_KC; kk += 16) {
                    acc[q] = __builtin_amdgcn_mfma_i32_32x32x16_i8(tb_load8(xi + kk), tb_load8(yj + kk), acc[q], 0, 0, 0);
                    acc[q] = __builtin_amdgcn_mfma_i32_32x32x16_i8(tb_load8(yi + kk), tb_load8(xj + kk), acc[q], 0, 0, 0);
                }
            }
        }
        // this phase's share of the row sums and diagonal terms
        u_acc += sx + sy;
        t_acc += dxy + 128 * (sx + sy) + 16384 * n;
    }
    if (t < (same ? 1 : 2) * TW_ROWS) {
        const int side = t / TW_ROWS, ri = t - side * TW_ROWS;
        (side ? U_j : U_i)[ri] = u_acc;
        (side ? T_j : T_i)[ri] = t_acc;
    }
    __syncthreads();
    const int *UJ = same ? U_i : U_j, *TJ = same ? T_i : T_j;

    // ---- epilogue: delta(i, j) for i < j of the wave's tiles
    const uint8_t *F = a.mats, *FT = F + (size_t)n * rs, *D = F + (size_t)2 * n * rs, *DT = F + (size_t)3 * n * rs;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (!has[q]) continue;
        const int jl = tJ[q] * 32 + (lane & 31), j = BJ * TW_ROWS + jl;
        if (j >= n) continue;
        const int pj = perm[j];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int il = tI[q] * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), i = BI * TW_ROWS + il;
            if (i < j) {
                const int pi = perm[i];
                const int s_ij = a.sym ? 2 * (acc[q][r] + 128 * (U_i[il] + UJ[jl]) + 32768 * n)
                                       : acc[q][r] + 128 * (U_i[il] + UJ[jl]) + 65536 * n;
                const int t_ii = a.sym ? 2 * T_i[il] : T_i[il], t_jj = a.sym ? 2 * TJ[jl] : TJ[jl];
                const int Dij = D[(size_t)i * rs + j], Dji = DT[(size_t)i * rs + j];
                const int Dii = D[(size_t)i * rs + i], Djj = D[(size_t)j * rs + j];
                const int Gij = F[(size_t)pi * rs + pj], Gji = FT[(size_t)pi * rs + pj];
                const int Gii = F[(size_t)pi * rs + pi], Gjj = F[(size_t)pj * rs + pj];
                const int c = -(Dji - Dii) * (Gii - Gji) - (Djj - Dij) * (Gij - Gjj) - (Dij - Dii) * (Gii - Gij)
                              - (Djj - Dji) * (Gji - Gjj) + (Dji - Dij) * (Gij - Gji) + (Djj - Dii) * (Gii - Gjj);
                out[pidx(n, i, j)] = s_ij - t_ii - t_jj + c;
            }
        }
    }
}


// The whole neighbourhood of one start, perm already in LDS (tb_plan layout at sm).
__device__ __attribute__((always_inline)) void table_mfma_body(const uint8_t *mats, int n, int sym, unsigned char *sm, int32_t *out) {
    const TbPlan P = tb_plan(n);
    const int grs = row_stride(n), rs = tb_stride(n), nr = (n + 15) & ~15, nt = tb_rows(n) / 32, L = blockDim.x,
              t = threadIdx.x;
    const int lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), half = lane >> 5, l5 = lane & 31;
    const int *perm = reinterpret_cast<const int *>(sm + P.perm);
    int *SD = reinterpret_cast<int *>(sm + P.sd), *DG = reinterpret_cast<int *>(sm + P.dg);
    int8_t *X = reinterpret_cast<int8_t *>(sm + P.x), *Y = reinterpret_cast<int8_t *>(sm + P.y);
    const int vpr = rs / 16;
    // 16 bytes of a global row less 128 (bytes past n stay zero)
    auto biased = [&](const uint8_t *row, int c) -> uint4 {
        uint4 x = *reinterpret_cast<const uint4 *>(row + c);
        unsigned m[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int real = n - (c + 4 * e);
            m[e] = real >= 4 ? 0x80808080u : (real <= 0 ? 0u : (0x80808080u >> (8 * (4 - real))));
        }
        return make_uint4(x.x ^ m[0], x.y ^ m[1], x.z ^ m[2], x.w ^ m[3]);
    };
    // rows of F into Y, X = F[p][p] gathered from them, then rows of D into Y
    for (int v = t; v < n * vpr; v += L) {
        const int i = v / vpr, c = (v - i * vpr) * 16;
        *reinterpret_cast<uint4 *>(Y + i * rs + c) = biased(mats + (size_t)i * grs, c);
    }
    __syncthreads();
    const int wpr = rs / 4;
    for (int v = t; v < nr * wpr; v += L) {
        const int i = v / wpr, k0 = (v - i * wpr) * 4;
        unsigned word = 0;
        if (i < n && k0 < n) {
            const uint8_t *row = reinterpret_cast<const uint8_t *>(Y) + perm[i] * rs;
            const int4 pk = *reinterpret_cast<const int4 *>(perm + k0);   // (entries past n: below)
            word = row[pk.x];
            if (k0 + 1 < n) word |= (unsigned)row[pk.y] << 8;
            if (k0 + 2 < n) word |= (unsigned)row[pk.z] << 16;
            if (k0 + 3 < n) word |= (unsigned)row[pk.w] << 24;
        }
        *reinterpret_cast<unsigned *>(X + i * rs + k0) = word;
    }
    __syncthreads();
    for (int v = t; v < nr * vpr; v += L) {
        const int i = v / vpr, c = (v - i * vpr) * 16;
        *reinterpret_cast<uint4 *>(Y + i * rs + c) =
            i < n ? biased(mats + ((size_t)2 * n + i) * grs, c) : make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    auto rows16 = [&](const int8_t *m, int row, int k) -> v4i { return *reinterpret_cast<const v4i *>(m + row * rs + k); };
    // 16 rows from row k of 16 columns from col (the lane's: col + l % 16), by transposing reads
    // of 8 rows; a lane addresses half a row of the 16 columns
    const int trow = (lane & 15) >> 1, tcol = (lane & 1) * 8;
    auto cols16 = [&](const int8_t *m, int k, int col) -> v4i {
        typedef __attribute__((address_space(3))) v2i *lds2;
        const v2i a = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds2)(m + (k + trow) * rs + col + tcol));
        const v2i b = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds2)(m + (k + trow + 8) * rs + col + tcol));
        return v4i{a[0], a[1], b[0], b[1]};
    };
    // T_ii and the diagonals, 32 indices a wave (entries past n are zero)
    if (w < nt) {
        const int i = w * 32 + l5, ic = min(i, n - 1);
        int td = 0;
        for (int k = 0; k < n; k += 16) {
            const v4i x = rows16(X, ic, k), y = rows16(Y, ic, k);
#pragma unroll
            for (int e = 0; e < 4; ++e) td = __builtin_amdgcn_sdot4(x[e], y[e], td, false);
            if (!sym) {
                const v4i xc = cols16(X, k, w * 32 + (lane & 16)), yc = cols16(Y, k, w * 32 + (lane & 16));
#pragma unroll
                for (int e = 0; e < 4; ++e) td = __builtin_amdgcn_sdot4(xc[e], yc[e], td, false);
            }
        }
        if (!half) {
            SD[i] = sym ? 2 * td : td;
            DG[i] = (int)(((unsigned)X[ic * rs + ic] << 16) | ((unsigned)Y[ic * rs + ic] & 0xffffu));
        }
    }
    __syncthreads();
    const int npairs = nt * (nt + 1) / 2;
    for (int pq = w; pq < npairs; pq += TB_W) {
        int I, J;
        tb_pair(pq, nt, I, J);
        v16i acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0;
        const int j = J * 32 + l5, jc = min(j, n - 1), ir = min(I * 32 + l5, n - 1);
        for (int k = 0; k < n; k += 32) {
            const int kk = min(k + half * 16, nr - 16);
            const bool in = k + half * 16 < n;
            v4i xi = rows16(X, ir, kk), yi = rows16(Y, ir, kk);
            v4i xj = rows16(X, jc, kk), yj = rows16(Y, jc, kk);
            if (!in) xi = yi = v4i{0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(xi, yj, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(yi, xj, acc, 0, 0, 0);
            if (!sym) {
                xi = cols16(X, kk, I * 32 + (lane & 16)), yi = cols16(Y, kk, I * 32 + (lane & 16));
                xj = cols16(X, kk, J * 32 + (lane & 16)), yj = cols16(Y, kk, J * 32 + (lane & 16));
                if (!in) xi = yi = v4i{0, 0, 0, 0};
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(xi, yj, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(yi, xj, acc, 0, 0, 0);
            }
        }
        // the rows of the lane's slots come four in a row: entries (j, i .. i + 3) are a word
        const int sj = SD[jc], gj = DG[jc];
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            const int i0 = I * 32 + 8 * y + 4 * half;
            const v4i si = *reinterpret_cast<const v4i *>(SD + i0), gi = *reinterpret_cast<const v4i *>(DG + i0);
            const int xw = *reinterpret_cast<const int *>(X + jc * rs + i0), yw = *reinterpret_cast<const int *>(Y + jc * rs + i0);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = i0 + e, ic = min(i, n - 1);
                const int g = (int)X[ic * rs + jc] + (int)(int8_t)(xw >> (8 * e)) - (gi[e] >> 16) - (gj >> 16);
                const int d = (int)Y[ic * rs + jc] + (int)(int8_t)(yw >> (8 * e)) - (int)(int16_t)gi[e] - (int)(int16_t)gj;
                const int a = acc[4 * y + e];
                if (i < j && j < n) out[pidx(n, i, j)] = (sym ? 2 * a : a) - si[e] - sj + __mul24(d, g);
            }
        }
    }
}

// table[j][idx(u,v)] for every start j of the launch.
__global__ void __launch_bounds__(TB_LANES) table_kernel(TableArgs a) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int bad;
    const TbPlan P = tb_plan(a.n);
    const int job = blockIdx.x, t = threadIdx.x;
    int32_t *out = a.table + (size_t)job * a.m;
    if (!tb_stage_perm(a.perms + (size_t)job * a.n, a.n, reinterpret_cast<int *>(sm + P.perm),
                       reinterpret_cast<int *>(sm + P.pinv), &bad)) {
        for (int i = t; i < a.m; i += blockDim.x) out[i] = 0;
        return;
    }
    table_mfma_body(a.mats, a.n, a.sym, sm, out);
}

// The neighbourhood of every item of a batch: block i takes item i's start.
__global__ void __launch_bounds__(TB_LANES) table_batch_kernel(BatchArgs b) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int bad;
    const Item &it = b.items[blockIdx.x];
    const TbPlan P = tb_plan(it.n);
    int32_t *out = b.table + it.table_off;
    if (!tb_stage_perm(b.perms + it.perm_off, it.n, reinterpret_cast<int *>(sm + P.perm),
                       reinterpret_cast<int *>(sm + P.pinv), &bad)) {
        for (int i = threadIdx.x; i < it.m; i += blockDim.x) out[i] = 0;
        return;
    }
    table_mfma_body(it.mats, it.n, it.sym, sm, out);
}

// Tables of starting items of a chunked run: block i writes items[i]'s neighbourhood
// into its `table`.
__global__ void __launch_bounds__(TB_LANES) table_items_kernel(const Item *items) {
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int bad;
    const Item &it = items[blockIdx.x];
    const TbPlan P = tb_plan(it.n);
    int32_t *out = const_cast<int32_t *>(it.table);
    if (!tb_stage_perm(it.perm_in, it.n, reinterpret_cast<int *>(sm + P.perm), reinterpret_cast<int *>(sm + P.pinv),
                       &bad)) {
        for (int i = threadIdx.x; i < it.m; i += blockDim.x) out[i] = 0;
        return;
    }
    table_mfma_body(it.mats, it.n, it.sym, sm, out);
}

size_t table_smem(int n) { return (size_t)tb_plan(n).total; }

size_t cost_smem(int n) { return (size_t)n * row_stride(n) + (size_t)2 * n * 4; }

}  // namespace

size_t table_smem_bytes(int n) { return table_smem(n); }

hipError_t launch_table_batch(const BatchArgs &b, size_t smem, hipStream_t st) {
    if (b.count <= 0) return hipSuccess;
    hipLaunchKernelGGL(table_batch_kernel, dim3(b.count), dim3(TB_LANES), smem, st, b);
    return report(hipGetLastError(), "batch table kernel launch");
}

hipError_t launch_table_items(const Item *d_items, int count, size_t smem, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(table_items_kernel, dim3(count), dim3(TB_LANES), smem, st, d_items);
    return report(hipGetLastError(), "item table kernel launch");
}

hipError_t launch_cost(const TableArgs &a, hipStream_t st) {
    if (a.k == 0) return hipSuccess;
    if (a.n > WIDE_N) {
        hipLaunchKernelGGL(cost_wide_kernel, dim3(a.k), dim3(256), (size_t)2 * a.n * 4, st, a);
        return report(hipGetLastError(), "kernel launch");
    }
    const size_t sm = cost_smem(a.n);
    hipLaunchKernelGGL(cost_kernel, dim3(a.k), dim3(256), sm, st, a);
    return report(hipGetLastError(), "kernel launch");
}

hipError_t launch_table(const TableArgs &a, hipStream_t st) {
    if (a.k == 0) return hipSuccess;
    if (a.n > WIDE_N) {   // starts in groups of at most 65535 (the grid's y extent)
        const int nb = (a.n + TW_ROWS - 1) / TW_ROWS;
        for (int j0 = 0; j0 < a.k; j0 += 65535) {
            TableArgs b = a;
            b.perms += (size_t)j0 * a.n;
            b.table += (size_t)j0 * a.m;
            b.k = a.k - j0 < 65535 ? a.k - j0 : 65535;
            hipLaunchKernelGGL(table_wide_mfma_kernel, dim3(nb * (nb + 1) / 2, b.k), dim3(TB_LANES),
                               (size_t)tw_plan(a.n).total, st, b);
            const hipError_t e = report(hipGetLastError(), "kernel launch");
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const size_t sm = table_smem(a.n);
    hipLaunchKernelGGL(table_kernel, dim3(a.k), dim3(TB_LANES), sm, st, a);
    return report(hipGetLastError(), "kernel launch");
}

}  // namespace qapk
