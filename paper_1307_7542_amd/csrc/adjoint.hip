// Adjoint of the Kronecker-sum product with respect to the model parameters.
//
// H depends linearly on every t_b, U_i and eps_i (Eq. count1 with per-bond and
// per-site parameters), so g^T (dH/dtheta) x is a bilinear form that reuses the
// structure of the product (Sec. IV A):
//   - bond b, spin up:   sum over entries (a, l) of H_up with bond b of
//                        (-esign) <g[a, :], x[l, :]>   (row dot products of V),
//   - bond b, spin down: sum over entries (b', l) of H_dn with bond b of
//                        (-esign) <g[:, b'], x[:, l]>  (column dot products),
//   - U_i:   sum_{a,b} n_i(up_a & dn_b) g[a,b] x[a,b],
//   - eps_i: sum_{a,b} (n_i(up_a) + n_i(dn_b)) g[a,b] x[a,b].
//
// No partial result per matrix entry goes through memory.  Spin up: a state has
// at most one hop per bond, so a table of partners [bond][state] (none where the
// bond's ends are equally occupied) lets a lane keep one accumulator per bond in
// registers, NB bonds at a time.  Spin down: the entries are uniform over a
// wavefront, which sums eight of them at a time over its lanes and adds them to
// its bond accumulators in LDS.  Every reduction has a fixed order (lanes
// over a fixed set of rows and columns, butterflies, in-order sums), so the
// result is reproducible.
#include <cmath>
#include <type_traits>
#include <vector>

#include "internal.h"

namespace hub {
namespace {

constexpr int NB = 32;  // bonds per launch (their accumulators are 64 registers)
constexpr uint32_t kNone = 0x7FFFFFFFu;

// -esign for a hop across bond (i < j) from state x: esign = (-1)^(occupied strictly between)
__device__ __forceinline__ bool esign_positive(uint32_t x, int i, int j)
{
    const uint32_t below_j = (j >= 32) ? 0xFFFFFFFFu : ((1u << j) - 1u);
    const uint32_t upto_i = (i >= 31) ? 0xFFFFFFFFu : ((1u << (i + 1)) - 1u);
    return (__popc(x & below_j & ~upto_i) & 1) == 0;
}

// Partner of every state across bonds e0 .. e0 + NB - 1, [NB][state]: {-esign <
// 0 : 1, basis index : 31}, kNone without a hop.
__global__ __launch_bounds__(256) void k_partners(int64_t count, const int32_t *__restrict__ rp,
                                                  const int32_t *__restrict__ col, const int32_t *__restrict__ bond,
                                                  const uint32_t *__restrict__ basis, const int32_t *__restrict__ bi,
                                                  const int32_t *__restrict__ bj, int e0, uint32_t *__restrict__ out)
{
    const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (a >= count) return;
    for (int e = 0; e < NB; ++e) out[e * count + a] = kNone;
    for (int k = rp[a]; k < rp[a + 1]; ++k) {
        const int e = bond[k] - e0;
        if (e < 0 || e >= NB) continue;
        out[e * count + a] =
            (uint32_t)col[k] | (esign_positive(basis[a], bi[e + e0], bj[e + e0]) ? 0x80000000u : 0u);
    }
}

// Every matrix entry as {-esign < 0 : 1, column : 31}, in CSR order
__global__ __launch_bounds__(256) void k_entries(int64_t count, const int32_t *__restrict__ rp,
                                                 const int32_t *__restrict__ col, const int32_t *__restrict__ bond,
                                                 const uint32_t *__restrict__ basis, const int32_t *__restrict__ bi,
                                                 const int32_t *__restrict__ bj, uint32_t *__restrict__ out)
{
    const int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (a >= count) return;
    for (int k = rp[a]; k < rp[a + 1]; ++k)
        out[k] = (uint32_t)col[k] | (esign_positive(basis[a], bi[bond[k]], bj[bond[k]]) ? 0x80000000u : 0u);
}

// The table of [NB][state] partners as pairs of bonds in one word, for columns
// that are staged whole: per half {-esign < 0 : 1, index : 15}, index = count
// without a hop (count <= 32767).
__global__ __launch_bounds__(256) void k_partner_pairs(int count, const uint32_t *__restrict__ part,
                                                       uint32_t *__restrict__ out)
{
    const int i = (int)blockIdx.x * 256 + threadIdx.x;
    const int e2 = (int)blockIdx.y;
    if (i >= count) return;
    uint32_t h[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint32_t p = part[(int64_t)(2 * e2 + u) * count + i];
        h[u] = p == kNone ? (uint32_t)count : (p & 0x7FFFu) | ((p >> 31) << 15);
    }
    out[(int64_t)e2 * count + i] = h[0] | (h[1] << 16);
}

__device__ __forceinline__ double wave_sum_a(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The sign of bit 31 of p applied to v.
__device__ __forceinline__ double signed_by(double v, uint32_t p)
{
    return __hiloint2double(__double2hiint(v) ^ (int)(p & 0x80000000u), __double2loint(v));
}

// Spin-up bonds: a workgroup takes columns in turn, stages rows [c0, c0 + n) of
// the x column in LDS (place n holds zero, for partners elsewhere or none) or, with
// long columns, gathers them from memory, and each lane adds g[a] x[partner] of its
// rows, `rows` of them from blockIdx.y on, to the bond's accumulator.
// Bound by the latency of the gathers, one per row and bond (half of them the
// broadcast zero), at three wavefronts a SIMD: on the 4x4 torus the LDS is busy 23 %
// of the cycles and the table comes from the L2 at 6.5 TB/s.  768 lanes: the
// accumulators spill at the 128 registers a lane has with 1024.
// GUARD: the zero place adds nothing, also where g[a] is infinite or NaN and its
// product with zero would be NaN (the form of a bond without a hop there); slower
// (4x4 torus 1.65 ms without), so run only when a first run's sums are not finite.
constexpr int UPB = 768;
enum UpMode { kPairs, kChunk, kGather };  // column staged whole (table of pairs), by chunks, or read from memory

template <int MODE, bool GUARD>
__global__ __launch_bounds__(UPB) void k_up_bonds(const double *__restrict__ g, const double *__restrict__ x, int cu,
                                                   int cd, int rows, int c0, int n, const uint32_t *__restrict__ part,
                                                   int nb, double *__restrict__ out)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double *xs = reinterpret_cast<double *>(smem_raw);
    double acc[NB];
#pragma unroll
    for (int e = 0; e < NB; ++e) acc[e] = 0.0;
    const int a_lo = (int)blockIdx.y * rows, a_hi = min(cu, a_lo + rows);
    for (int b = blockIdx.x; b < cd; b += gridDim.x) {
        const double *__restrict__ xb = x + (int64_t)b * cu + c0, *__restrict__ gb = g + (int64_t)b * cu;
        if (MODE != kGather) {
            for (int a = threadIdx.x; a < n; a += UPB) xs[a] = xb[a];
            if (threadIdx.x == 0) xs[n] = 0.0;
            __syncthreads();
        }
        for (int a = a_lo + (int)threadIdx.x; a < a_hi; a += UPB) {
            const double ga = gb[a];
            if (MODE == kPairs) {
#pragma unroll
                for (int e8 = 0; e8 < NB; e8 += 8) {
                    if (e8 >= nb) break;
                    uint32_t p[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) p[u] = part[(int64_t)(e8 / 2 + u) * cu + a];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t a0 = p[u] & 0x7FFFu, a1 = (p[u] >> 16) & 0x7FFFu;
                        const double v0 = xs[a0], v1 = xs[a1];
                        const double g0 = GUARD && a0 == (uint32_t)n ? 0.0 : ga, g1 = GUARD && a1 == (uint32_t)n ? 0.0 : ga;
                        acc[e8 + 2 * u] = fma(signed_by(g0, p[u] << 16), v0, acc[e8 + 2 * u]);
                        acc[e8 + 2 * u + 1] = fma(signed_by(g1, p[u]), v1, acc[e8 + 2 * u + 1]);
                    }
                }
                continue;
            }
#pragma unroll
            for (int e8 = 0; e8 < NB; e8 += 8) {
                if (e8 >= nb) break;
                uint32_t p[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) p[u] = part[(int64_t)min(e8 + u, nb - 1) * cu + a];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (MODE == kGather) {  // no partner: the lane's own row instead, and nothing added
                        const bool none = (p[u] & kNone) == kNone;
                        const double v = xb[none ? (uint32_t)a : p[u] & kNone];
                        const double sum = fma(signed_by(ga, p[u]), v, acc[e8 + u]);
                        acc[e8 + u] = none ? acc[e8 + u] : sum;
                        continue;
                    }
                    const uint32_t at = min((p[u] & kNone) - (uint32_t)c0, (uint32_t)n);
                    const double v = xs[at], gu = GUARD && at == (uint32_t)n ? 0.0 : ga;
                    acc[e8 + u] = fma(signed_by(gu, p[u]), v, acc[e8 + u]);
                }
            }
        }
        if (MODE != kGather) __syncthreads();
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int e = 0; e < NB; ++e) {
        const double r = wave_sum_a(acc[e]);
        if (lane == 0 && e < nb) xs[wave * NB + e] = r;
    }
    __syncthreads();
    if ((int)threadIdx.x < nb) {
        double r = 0.0;
#pragma unroll
        for (int w = 0; w < UPB / 64; ++w) r += xs[w * NB + threadIdx.x];
        out[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * NB + threadIdx.x] = r;
    }
}

// Rows r0, r0 + 1 of a column; FULL: both inside it, else zero from row cu on.
template <bool FULL>
__device__ __forceinline__ double2 ld_rows(const double *__restrict__ col, int r0, int cu)
{
    typedef double VecU __attribute__((ext_vector_type(2), aligned(8)));
    if (FULL) {
        const VecU v = *reinterpret_cast<const VecU *>(col + r0);
        return make_double2(v[0], v[1]);
    }
    return make_double2(r0 < cu ? col[r0] : 0.0, r0 + 1 < cu ? col[r0 + 1] : 0.0);
}

// v of another lane of the same row of 16, chosen by the DPP control C
template <int C>
__device__ __forceinline__ double dpp(double v)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), C, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), C, 0xf, 0xf, false));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kRor4 = 0x124, kRor8 = 0x128;  // quad_perm, row_ror (8: xor 8)

// Entry of eight whose sum wave_sum8 leaves in lane l (the same in lanes that differ in bits 2, 3, 5)
__device__ __forceinline__ int wave_sum8_entry(int l) { return (l & 3) | ((l >> 2) & 4); }

// The sums over the wavefront of eight values per lane; lanes keep half of the
// values in each of three exchanges, so that one value is left to add up.
__device__ __forceinline__ double wave_sum8(const double (&p)[8], int lane)
{
    double a[4], b[2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        a[i] = ((lane & 1) ? p[2 * i + 1] : p[2 * i]) + dpp<kXor1>((lane & 1) ? p[2 * i] : p[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 2; ++i)
        b[i] = ((lane & 2) ? a[2 * i + 1] : a[2 * i]) + dpp<kXor2>((lane & 2) ? a[2 * i] : a[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) {  // over the row of 16 lanes: xor 8, then 4
        b[i] += dpp<kRor8>(b[i]);
        b[i] += dpp<kRor4>(b[i]);
    }
    double c = ((lane & 16) ? b[1] : b[0]) + __shfl_xor((lane & 16) ? b[0] : b[1], 16, 64);
    c += __shfl_xor(c, 32, 64);
    return c;
}

// slot[bond of entry] += -esign <g[:, b], x[:, column of entry]> over rows r0, r0 +
// 1 of columns b0, b0 + step, ... < cd, by one wavefront
template <bool FULL>
__device__ __forceinline__ void dn_columns(double *slot, const double *__restrict__ g, const double *__restrict__ x,
                                           int cu, int cd, int r0, int b0, int step, const int32_t *__restrict__ rp,
                                           const uint32_t *__restrict__ ent, const int32_t *__restrict__ bond, int lane)
{
    for (int b = b0; b < cd; b += step) {
        const double2 gv = ld_rows<FULL>(g + (int64_t)b * cu, r0, cu);
        const int ks = rp[b], n = rp[b + 1] - ks;
        const uint32_t *__restrict__ e = ent + ks;
        const int lu = wave_sum8_entry(lane);
        for (int k = 0; k < n; k += 8) {
            const int m = min(8, n - k);
            const bool mine = (lane & 44) == 0 && lu < m;
            const int bd = mine ? bond[ks + k + lu] : 0;
            const uint32_t es = mine ? e[k + lu] : 0u;
            double2 v[8];
            if (m == 8) {
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    v[u] = ld_rows<FULL>(x + (uint64_t)(e[k + u] & kNone) * (uint32_t)cu, r0, cu);
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    v[u] = make_double2(0.0, 0.0);
                    if (u < m) v[u] = ld_rows<FULL>(x + (uint64_t)(e[k + u] & kNone) * (uint32_t)cu, r0, cu);
                }
            }
            double p[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) p[u] = fma(gv.x, v[u].x, gv.y * v[u].y);
            const double r = wave_sum8(p, lane);
            if (mine) slot[bd] += (es & 0x80000000u) ? -r : r;
        }
    }
}

// Spin-down bonds: a segment of 128 rows belongs to 4 ntile wavefronts that take
// its columns in turn, so that together they sweep the columns in order (ordered
// by segment, an eighth per XCD, as k_dn_rows of the product); slots [nb] per
// wavefront in LDS (the bonds of a column's entries are distinct).  Bound as
// k_dn_rows by the lines in flight: a segment has as many workgroups as an XCD
// runs at a time, so that they all read one band of rows out of its L2.
__global__ __launch_bounds__(256) void k_dn_bonds(const double *__restrict__ g, const double *__restrict__ x, int cu,
                                                  int cd, int ntile, int nwork, const int32_t *__restrict__ rp,
                                                  const uint32_t *__restrict__ ent, const int32_t *__restrict__ bond,
                                                  int nb, double *__restrict__ out)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int per = (nwork + 7) >> 3;
    const int blk = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    if ((int)(blockIdx.x >> 3) >= per || blk >= nwork) return;
    double *slot = reinterpret_cast<double *>(smem_raw) + w * nb;
    for (int e = lane; e < nb; e += 64) slot[e] = 0.0;
    const int seg = (int)((uint32_t)blk / (uint32_t)ntile), tile = blk - seg * ntile;
    const int r0 = seg * 128 + 2 * lane, b0 = tile * 4 + w, step = 4 * ntile;
    if (seg * 128 + 128 <= cu) dn_columns<true>(slot, g, x, cu, cd, r0, b0, step, rp, ent, bond, lane);
    else dn_columns<false>(slot, g, x, cu, cd, r0, b0, step, rp, ent, bond, lane);
    __syncthreads();
    const double *all = reinterpret_cast<const double *>(smem_raw);
    for (int e = threadIdx.x; e < nb; e += 256)
        out[(int64_t)blk * nb + e] = (all[e] + all[nb + e]) + (all[2 * nb + e] + all[3 * nb + e]);
}

// Site forms: a wavefront takes columns in turn; over a column its lanes sum t_i
// = sum_a n_i(a) g x and s = sum_a g x, and the column's bits are uniform:
// U_i gets n_i(b) t_i, eps_i gets t_i + n_i(b) s.  Both vectors once, 3.6 TB/s on the
// 4x4 torus: 40 lines in flight per CU at 789 cycles each.
template <int MM>
__global__ __launch_bounds__(256) void k_site_terms(const double *__restrict__ g, const double *__restrict__ x, int cu,
                                                    int cd, int rows, int M, const uint32_t *__restrict__ up,
                                                    const uint32_t *__restrict__ dn, double *__restrict__ out)
{
    const int lane = threadIdx.x & 63;
    const int wave = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lo = (int)blockIdx.y * rows, hi = min(cu, lo + rows);
    double aU[MM], aE[MM];
#pragma unroll
    for (int i = 0; i < MM; ++i) aU[i] = aE[i] = 0.0;
    for (int b = wave; b < cd; b += (int)gridDim.x * 4) {
        const double *__restrict__ gb = g + (int64_t)b * cu, *__restrict__ xb = x + (int64_t)b * cu;
        double t[MM], s = 0.0;
#pragma unroll
        for (int i = 0; i < MM; ++i) t[i] = 0.0;
        for (int r = lo; r < hi; r += 256) {
            double gx[4];
            uint32_t ua[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int a = r + u * 64 + lane;
                gx[u] = a < hi ? gb[a] * xb[a] : 0.0;
                ua[u] = a < hi ? up[a] : 0u;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                s += gx[u];
#pragma unroll
                for (int i = 0; i < MM; ++i) t[i] += ((ua[u] >> i) & 1u) ? gx[u] : 0.0;
            }
        }
        const uint32_t db = dn[b];
#pragma unroll
        for (int i = 0; i < MM; ++i) {
            aE[i] += t[i];
            if ((db >> i) & 1u) {
                aU[i] += t[i];
                aE[i] += s;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < MM; ++i) {
        const double rU = wave_sum_a(aU[i]), rE = wave_sum_a(aE[i]);
        if (lane == 0 && i < M) {
            double *o = out + ((int64_t)blockIdx.y * gridDim.x * 4 + wave) * 2 * kMaxSites;
            o[i] = rU;
            o[kMaxSites + i] = rE;
        }
    }
}

// out[j] (+)= sum over rows r of part[r * stride + j], one workgroup per j, in a fixed order
__global__ __launch_bounds__(1024) void k_column_sum(const double *__restrict__ part, int64_t rows, int stride,
                                                     double *__restrict__ out, int add)
{
    __shared__ double s[16];
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    const double *__restrict__ p = part + blockIdx.x;
    int64_t r = threadIdx.x;
    for (; r + 3 * 1024 < rows; r += 4 * 1024)
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] += p[(r + u * 1024) * stride];
    for (; r < rows; r += 1024) a[0] += p[r * stride];
    const double acc = wave_sum_a((a[0] + a[1]) + (a[2] + a[3]));
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 16; ++w) t += s[w];
        out[blockIdx.x] = add ? out[blockIdx.x] + t : t;
    }
}

hub_status allow_up_lds(size_t bytes)
{
    for (const void *k : {(const void *)k_up_bonds<kPairs, false>, (const void *)k_up_bonds<kChunk, false>,
                          (const void *)k_up_bonds<kPairs, true>, (const void *)k_up_bonds<kChunk, true>})
        HUB_HIP(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    return HUB_OK;
}

}  // namespace

hub_status param_bilinear(const hub_sector *s, const double *g, const double *x, double *dbond, double *dU,
                          double *deps, hipStream_t st)
{
    const SpinTables &U = s->spin[0];
    const SpinTables &D = s->spin[1];
    const int cu = (int)U.count, cd = (int)D.count, M = s->M, nb = s->nb;
    // `want` workgroups over columns and, where these are fewer, parts of the rows
    // of at least `least` (one column of 2704156 rows: 1027 ms on one workgroup, by
    // chunks, 12.7 ms on all of them, 0.67 gathered)
    auto row_part = [&](int columns, int want, int least) {
        const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(want / columns, cu / least));
        return (int)(((cu + parts - 1) / parts + 255) / 256 * 256);
    };
    // site forms: 4 wavefronts a workgroup, at most 8 workgroups per CU
    const int site_cols = (int)std::min<int64_t>((cd + 3) / 4, 2048);
    const int site_rows = row_part(site_cols, 2048, 1024), site_parts = (cu + site_rows - 1) / site_rows;
    const int64_t site_grid = (int64_t)site_cols * site_parts;
    // spin-up bonds: one workgroup per CU or two, each with its share of the columns
    const size_t lds = s->lds_max;
    const int chunk = (int)std::min<int64_t>(cu, (int64_t)(lds / sizeof(double)) - 1);
    const int chunks = (cu + chunk - 1) / chunk;
    // Chunks cost a pass over the whole table and every row each; from three on x is
    // gathered from memory instead, 20-site ring with 10 + 1 electrons (10 chunks)
    // 905 -> 222 us, 2x9 ladder with 9 + 3 (3 chunks) 2.58 -> 2.09 ms.  With two the
    // chunks are better where it counts: 2x9 ladder with 7 + 7 42.6 against 49.3 ms
    // (17-site ring with 8 + 7 16.0 against 15.2).
    const int mode = chunks >= 3 ? kGather : chunks == 1 && cu <= 32767 ? kPairs : kChunk;
    const int up_cols = std::min(cd, 512);
    const int up_rows = row_part(up_cols, 512, 4 * UPB), up_parts = (cu + up_rows - 1) / up_rows;
    const int64_t up_grid = (int64_t)up_cols * up_parts;
    const size_t up_lds = std::max<size_t>(mode == kGather ? 0 : (size_t)chunk + 1, (UPB / 64) * NB) * sizeof(double);
    // spin-down bonds: workgroups per segment of 128 rows (k_dn_bonds)
    const int nseg = (cu + 127) / 128;
    // (fewer where a launch of 256 lanes each would not hold them: below 2^24 in all)
    const int ntile = std::min(std::min((cd + 3) / 4, 256), ((1 << 24) - 8) / nseg);
    const int64_t nwork = (int64_t)nseg * ntile;

    Workspace mem(st);
    double *res = nullptr, *site = nullptr, *pu = nullptr, *pd = nullptr;  // res: bonds, then U and eps forms
    uint32_t *tu = nullptr, *td = nullptr, *tp = nullptr;
    const int nres = nb + 2 * kMaxSites;
    HUB_TRY(mem.alloc((void **)&res, sizeof(double) * (size_t)nres));
    HUB_TRY(mem.alloc((void **)&site, sizeof(double) * (size_t)site_grid * 4 * 2 * kMaxSites));
    if (nb > 0) {
        HUB_TRY(mem.alloc((void **)&pu, sizeof(double) * (size_t)up_grid * NB));
        HUB_TRY(mem.alloc((void **)&pd, sizeof(double) * (size_t)nwork * (size_t)nb));
        HUB_TRY(mem.alloc((void **)&tu, sizeof(uint32_t) * (size_t)cu * NB));
        HUB_TRY(mem.alloc((void **)&td, sizeof(uint32_t) * (size_t)std::max<int64_t>(D.nnz, 1)));
        if (mode == kPairs) HUB_TRY(mem.alloc((void **)&tp, sizeof(uint32_t) * (size_t)cu * (NB / 2)));
        HUB_TRY(allow_up_lds(lds));
    }
#define HUB_SITE(MMV)                                                                                           \
    hipLaunchKernelGGL(k_site_terms<MMV>, dim3(site_cols, site_parts), dim3(256), 0, st, g, x, cu, cd, site_rows, M,    \
                       U.basis, D.basis, site)
    if (M <= 8) HUB_SITE(8);
    else if (M <= 16) HUB_SITE(16);
    else if (M <= 24) HUB_SITE(24);
    else HUB_SITE(32);
#undef HUB_SITE
    hipLaunchKernelGGL(k_column_sum, dim3(2 * kMaxSites), dim3(1024), 0, st, (const double *)site,
                       site_grid * 4, 2 * kMaxSites, res + nb, 0);
    if (nb > 0) {
        hipLaunchKernelGGL(k_entries, dim3((cd + 255) / 256), dim3(256), 0, st, (int64_t)cd, D.rp, D.col, D.bond,
                           D.basis, s->d_bi, s->d_bj, td);
        hipLaunchKernelGGL(k_dn_bonds, dim3((unsigned)(8 * ((nwork + 7) / 8))), dim3(256), 4 * nb * sizeof(double), st,
                           g, x, cu, cd, ntile, (int)nwork, D.rp, (const uint32_t *)td, D.bond, nb, pd);
    }
    std::vector<double> h((size_t)nres);
    auto bonds = [&](auto guard) -> hub_status {
        constexpr bool G = decltype(guard)::value;
        if (nb > 0)
            hipLaunchKernelGGL(k_column_sum, dim3(nb), dim3(1024), 0, st, (const double *)pd, nwork, nb, res, 0);
        for (int e0 = 0; e0 < nb; e0 += NB) {
            const int n = std::min(NB, nb - e0);
            hipLaunchKernelGGL(k_partners, dim3((cu + 255) / 256), dim3(256), 0, st, (int64_t)cu, U.rp, U.col, U.bond,
                               U.basis, s->d_bi, s->d_bj, e0, tu);
            if (mode == kPairs)
                hipLaunchKernelGGL(k_partner_pairs, dim3((cu + 255) / 256, NB / 2), dim3(256), 0, st, cu,
                                   (const uint32_t *)tu, tp);
            for (int c0 = 0; c0 < cu; c0 += mode == kGather ? cu : chunk) {
                const uint32_t *table = mode == kPairs ? tp : tu;
                auto run = [&](auto kernel) {
                    hipLaunchKernelGGL(kernel, dim3(up_cols, up_parts), dim3(UPB), up_lds, st, g, x, cu, cd, up_rows, c0,
                                       std::min(chunk, cu - c0), table, n, pu);
                };
                if (mode == kGather) run(k_up_bonds<kGather, false>);
                else if (mode == kPairs) run(k_up_bonds<kPairs, G>);
                else run(k_up_bonds<kChunk, G>);
                hipLaunchKernelGGL(k_column_sum, dim3(n), dim3(1024), 0, st, (const double *)pu, up_grid, NB, res + e0,
                                   1);
            }
        }
        HUB_HIP(hipGetLastError());
        HUB_HIP(hipMemcpyAsync(h.data(), res, sizeof(double) * h.size(), hipMemcpyDeviceToHost, st));
        HUB_HIP(hipStreamSynchronize(st));
        return HUB_OK;
    };
    HUB_TRY(bonds(std::false_type{}));
    bool finite = true;
    for (int b = 0; b < nb; ++b) finite = finite && std::isfinite(h[(size_t)b]);
    if (!finite) HUB_TRY(bonds(std::true_type{}));
    for (int b = 0; dbond && b < nb; ++b) dbond[b] = h[(size_t)b];
    for (int i = 0; i < M; ++i) {
        if (dU) dU[i] = h[(size_t)nb + i];
        if (deps) deps[i] = h[(size_t)nb + kMaxSites + i];
    }
    return HUB_OK;
}

}  // namespace hub
