// a5 / a6: paged decode attention over the variable-budget Cascade Cache, and the
// append-only dense-tier write of one decode step (gfx950).
//
// Decode (App. F): every (sequence, KV head) is split into ranges of pages; a workgroup
// computes the attention state (o, m, l) of the G query heads of that KV head over its
// range (each K/V page is read once for all G heads: head expansion), and a merge kernel
// combines the ranges with the merge operator
//   o(I u J) = (o(I) SE(I) + o(J) SE(J)) / (SE(I) + SE(J)),  SE(I u J) = SE(I) + SE(J).
// Only pages below n_pages are visited and page masks drop invalid slots, so the work
// follows each head's own budget: a row's pages are shared by the launch's splits, a split
// past the row's end exits at once, and the merge reads only the splits that held pages.
// Each split stages its page ids and masks in LDS, and every wave keeps the next page's
// loads in flight while it computes the current one.
//
// bf16 caches run on the matrix cores (decode_split_kernel); fp32 caches on the VALU, one page
// per wave at a time (decode_split_f32_kernel), with this lane mapping:
//   scores  lane = 4 * t + c: slot t, quarter c of the head dimension; partial dot
//           products are summed over the 4 lanes of a slot with two xor-shuffles;
//   values  lane = LPR * kg + dc: 16-byte chunk dc of the row, slots kg*KPL .. +KPL;
//           the probabilities reach those lanes by shuffles.
#include <mutex>
#include <type_traits>

#include "hk_internal.h"
#include "hk_turn.h"

namespace hk {

constexpr int DEC_NT = 256;                 // threads per workgroup
constexpr int DEC_NW = DEC_NT / 64;
constexpr int DEC_PPS = 128;                // most pages per split (one workgroup)
constexpr int DEC_PPS_MIN = 16;             // fewest pages per split
constexpr int DEC_TARGET_WG = 2048;         // workgroups a launch should offer the chip

// Pages per split for a row of n pages: the row is shared evenly by the launch's n_split
// splits, at least DEC_PPS_MIN pages each and at most pps (never above DEC_PPS).  Split i
// covers pages [i * share, min((i + 1) * share, n)); the splits with i * share >= n hold
// nothing, write nothing, and the merge reads only the ceil(n / share) splits before them.
__device__ __forceinline__ int decode_share(int n, int n_split, int pps) {
  return min(min(pps, DEC_PPS), max((n + n_split - 1) / n_split, DEC_PPS_MIN));
}

template <int D, int G>
__global__ __launch_bounds__(DEC_NT) void decode_split_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k_pool, const float* __restrict__ v_pool,
    const int32_t* __restrict__ table, const uint16_t* __restrict__ masks,
    const int32_t* __restrict__ n_pages_arr, int Hq, int Hkv, int max_pages, float c2,
    float* __restrict__ part, int n_split, int pps) {
  constexpr int ES = sizeof(float);
  constexpr int DQ = D / 4;                 // dims per quarter
  constexpr int VEC = 16 / ES;              // elements per 16-byte chunk
  constexpr int LPR = D / VEC;              // lanes per value row
  constexpr int KG = 64 / LPR;              // slot groups
  constexpr int KPL = HK_PAGE / KG;         // slots per lane (values)
  constexpr int QW = DQ * ES / 4;           // 32-bit words of the query quarter
  __shared__ float s_m[DEC_NW][G], s_l[DEC_NW][G];
  __shared__ float s_o[DEC_NW][G][D];

  const int h = blockIdx.y, split = blockIdx.x;
  const int s = h / Hkv, kv = h % Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = min(n_pages_arr[h], max_pages);
  // this head's pages are shared evenly by the launch's splits, so short rows are not left
  // to few waves; a split past the row's end leaves at once (the merge skips it)
  const int per = decode_share(n, n_split, pps);
  const int p_begin = split * per, p_end = min(p_begin + per, n);
  if (p_begin >= n) return;
  const int t = lane >> 2, c = lane & 3;
  const int kg = lane / LPR, dc = lane % LPR;

  // the G query rows of this KV head (contiguous in q), 16 bytes per thread
  __shared__ uint4 s_q[G * D * ES / 16];
  {
    const uint4* src = reinterpret_cast<const uint4*>(q + ((size_t)s * Hq + kv * G) * D);
    for (int i = threadIdx.x; i < G * D * ES / 16; i += DEC_NT) s_q[i] = src[i];
  }
  // the split's page ids and masks, staged once: a page's loads then wait on no global
  // read of the table (the per-share bound above keeps the range within DEC_PPS)
  const int32_t* trow = table + (size_t)h * max_pages;
  const uint16_t* mrow = masks + (size_t)h * max_pages;
  __shared__ int32_t s_pid[DEC_PPS];
  __shared__ uint16_t s_pm[DEC_PPS];
  for (int i = threadIdx.x; i < p_end - p_begin; i += DEC_NT) {
    s_pid[i] = trow[p_begin + i];
    s_pm[i] = mrow[p_begin + i];
  }
  __syncthreads();
  const int q_lane = c * DQ * ES / 16;
  auto q_word = [&](int qb, int g, int i) -> uint32_t {
    const uint4 u = s_q[qb + g * D * ES / 16 + i / 4];
    return (i & 3) == 0 ? u.x : (i & 3) == 1 ? u.y : (i & 3) == 2 ? u.z : u.w;
  };
  float m_run[G], l_part[G], o[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m_run[g] = -INFINITY;
    l_part[g] = 0.f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) o[g][e] = 0.f;
  }
  struct PageRegs {
    uint4 k[QW / 4];
    uint4 v[KPL];
    uint32_t m16;
  };
  // the wave's pages are p_begin + wave + DEC_NW * j, j < npg; load_page(r, j) reads
  // page min(j, npg - 1) and gives it an empty mask when j >= npg
  const int npg = p_begin + wave < p_end ? (p_end - 1 - p_begin - wave) / DEC_NW + 1 : 0;
  auto load_page = [&](PageRegs& r, int j) {
    const int li = wave + DEC_NW * min(j, npg - 1);
    r.m16 = j < npg ? s_pm[li] : 0u;
    const size_t page = (size_t)s_pid[li] * HK_PAGE;
    const uint4* ks = reinterpret_cast<const uint4*>(k_pool + (page + t) * D + c * DQ);
#pragma unroll
    for (int i = 0; i < QW / 4; ++i) r.k[i] = ks[i];
#pragma unroll
    for (int i = 0; i < KPL; ++i)
      r.v[i] = *reinterpret_cast<const uint4*>(v_pool + (page + kg * KPL + i) * D + dc * VEC);
  };
  auto process_page = [&](const PageRegs& r) {
    const uint32_t m16 = r.m16;
    uint32_t kw[QW];
#pragma unroll
    for (int i = 0; i < QW / 4; ++i) {
      kw[4 * i + 0] = r.k[i].x;
      kw[4 * i + 1] = r.k[i].y;
      kw[4 * i + 2] = r.k[i].z;
      kw[4 * i + 3] = r.k[i].w;
    }
    const bool valid = (m16 >> t) & 1u;
    // the query words are read from LDS for every page (an opaque offset keeps the
    // compiler from hoisting them into 64 more registers per lane)
    int qb = q_lane;
    asm volatile("" : "+v"(qb));
    float zl[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float z = 0.f;
#pragma unroll
      for (int i = 0; i < QW; ++i) z = fmaf(__uint_as_float(q_word(qb, g, i)), __uint_as_float(kw[i]), z);
      z += __shfl_xor(z, 1, 64);
      z += __shfl_xor(z, 2, 64);
      zl[g] = valid ? z * c2 : -INFINITY;      // log2 units
    }
    float pr[G], alpha[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      // the 4 lanes of a slot hold the same value, so within a 16-lane row the half-row
      // and row mirrors (lane l <-> 7 - l within 8, l <-> 15 - l) meet every slot of the row
      float pm = zl[g];
      pm = fmaxf(pm, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                         0, __builtin_bit_cast(int, pm), 0x141, 0xf, 0xf, false)));
      pm = fmaxf(pm, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                         0, __builtin_bit_cast(int, pm), 0x140, 0xf, 0xf, false)));
      pm = fmaxf(pm, __shfl_xor(pm, 16, 64));
      pm = fmaxf(pm, __shfl_xor(pm, 32, 64));
      // a page with no valid slot leaves the state as it is (alpha 1 or the state still
      // empty, pr 0); the guards keep -inf - -inf out of the exponentials
      const float mn = fmaxf(m_run[g], pm);
      alpha[g] = m_run[g] == -INFINITY ? 0.f : fast_exp2(m_run[g] - mn);
      pr[g] = valid ? fast_exp2(zl[g] - mn) : 0.f;
      m_run[g] = mn;
      l_part[g] = l_part[g] * alpha[g] + (c == 0 ? pr[g] : 0.f);
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < VEC; ++e) o[g][e] *= alpha[g];
#pragma unroll
    for (int i = 0; i < KPL; ++i) {
      const int src_lane = 4 * (kg * KPL + i);
      float vf[VEC];
      const uint32_t vv[4] = {r.v[i].x, r.v[i].y, r.v[i].z, r.v[i].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) vf[e] = __uint_as_float(vv[e]);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float pg = __shfl(pr[g], src_lane, 64);
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[g][e] = fmaf(pg, vf[e], o[g][e]);
      }
    }
  };

  // the wave's next page is loaded (into the other register set) before the current one
  // is processed; the loop is unrolled by two so both sets stay in registers.  Every
  // trip issues both loads and processes both sets (a page past the wave's run is its
  // last page again with an empty mask, which leaves the state as it is), so no load is
  // moved behind the processing it should overlap.
  if (npg > 0) {
    PageRegs ra, rb;
    load_page(ra, 0);
    for (int j = 0; j < npg; j += 2) {
      load_page(rb, j + 1);
      process_page(ra);
      load_page(ra, j + 2);
      process_page(rb);
    }
  }
  // reduce over slot groups (lanes with the same value chunk) and over all lanes for l
#pragma unroll
  for (int g = 0; g < G; ++g) {
#pragma unroll
    for (int x = LPR; x < 64; x <<= 1)
#pragma unroll
      for (int e = 0; e < VEC; ++e) o[g][e] += __shfl_xor(o[g][e], x, 64);
    l_part[g] = wave_sum(l_part[g]);
    if (lane == 0) {
      s_m[wave][g] = m_run[g];
      s_l[wave][g] = l_part[g];
    }
    if (lane < LPR)
#pragma unroll
      for (int e = 0; e < VEC; ++e) s_o[wave][g][dc * VEC + e] = o[g][e];
  }
  __syncthreads();
  // combine the waves -> one partial state per (head, split, g): [o(D) unnormalised, m, l]
  for (int idx = threadIdx.x; idx < G * D; idx += DEC_NT) {
    const int g = idx / D, d = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < DEC_NW; ++w) M = fmaxf(M, s_m[w][g]);
    float L = 0.f, O = 0.f;
    if (M != -INFINITY)
#pragma unroll
      for (int w = 0; w < DEC_NW; ++w) {
        const float a = fast_exp2(s_m[w][g] - M);
        L += s_l[w][g] * a;
        O += s_o[w][g][d] * a;
      }
    float* dst = part + (((size_t)h * n_split + split) * G + g) * (D + 2);
    dst[d] = O;
    if (d == 0) {
      dst[D] = M;
      dst[D + 1] = L;
    }
  }
}

// ------------------------------------------------------------------ bf16 caches: matrix cores
// The same split on MFMA 16x16x32, for any group of up to 8 query heads.  A wave takes two pages
// (32 keys) at a time:
//   scores  C[key][query] = K Q^T, one 16x16 tile per page: lane l supplies key l % 16 and dims
//           32 s + 8 (l / 16) .. +8 of step s, and holds, of query l % 16, the keys 4 (l / 16) + r;
//   values  C[query][dim] += P V: the contraction runs over the 32 keys in the order in which
//           the score tiles leave them, so a lane's own 8 probabilities are its A operand and no
//           probability crosses lanes.  A lane loads the 16-byte (D 64: 8-byte) piece l % 16 of
//           the V rows of those 8 keys; two v_perm per pair of words turn rows into columns.
// K of the next pair is requested as soon as the scores have read this pair's, V after its
// columns are formed: one pair's registers, always full.  The usual pair needs no cross-lane
// maximum: the running reference m moves only when a score exceeds it by 2^DEC_SLACK (the
// merge takes any reference).
// Precision.  P keeps its 24 bits: it is split exactly into three bf16 parts, whose products
// with V are exact.  A pair's sum is formed by three MFMAs from zero and added to the running
// sum by a rounded fp32 add.  The matrix cores cut sums downward, a bias that grew with the row
// (3.4e-7 of the result at 65536 keys against 2.3e-7 for the VALU form): every other pair is
// formed with the opposite sign and counted back, and a score is the sum of two shorter chains.
// m is a whole number, so every rescaling factor of the state and of the merges is an exact
// power of two.  Error of o against 64 bits, VALU form -> this: 1.77 -> 1.53e-7 (rows of 2000),
// 2.41 -> 1.74e-7 (8192), 2.10 -> 1.91e-7 (23k to 33k), 2.31 -> 2.14e-7 (33k to 66k).
// Bound by HBM reads.  The VALU form (two pages of prefetch, fdot2 and per-head fma) was
// bound by issue from 7 heads on: 512 heads x 8 x 3000 tokens 218 -> 161 us, 512 x 4 x 8192 378 ->
// 370 (5.8 TB/s), 512 x 4 x 800-5600 172 -> 164, 512 x 1 x 8192 unchanged at 359; 16 x 7 x 23k to 33k
// 80 -> 56, both with the merge as it is.
constexpr float DEC_SLACK = 16.f;
constexpr int DEC_GMAX = 8;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int D>
__global__ __launch_bounds__(DEC_NT) __attribute__((amdgpu_waves_per_eu(3, 4))) void decode_split_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_pool, const uint16_t* __restrict__ v_pool,
    const int32_t* __restrict__ table, const uint16_t* __restrict__ masks,
    const int32_t* __restrict__ n_pages_arr, int G, int Hq, int Hkv, int max_pages, float c2,
    float* __restrict__ part, int n_split, int pps, uint32_t heads_first) {
  constexpr int KS = D / 32;                // MFMA steps over the head dimension
  constexpr int VE = D / 16;                // dims of a V piece
  constexpr int VW = VE / 2;                // 32-bit words of a V piece
  using vpiece = std::conditional_t<VW == 4, u32x4, u32x2>;
  __shared__ float s_m[DEC_NW][DEC_GMAX], s_l[DEC_NW][DEC_GMAX];
  __shared__ __align__(16) float s_o[DEC_NW][DEC_GMAX][D];
  __shared__ int32_t s_pid[DEC_PPS];
  __shared__ uint16_t s_pm[DEC_PPS];

  int h = blockIdx.y, split = blockIdx.x;
  if (heads_first) {
    split = h;
    h = head_of(blockIdx.x, split, (int)gridDim.x, heads_first);
  }
  const int s = h / Hkv, kv = h % Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = min(n_pages_arr[h], max_pages);
  const int per = decode_share(n, n_split, pps);
  const int p_begin = split * per, p_end = min(p_begin + per, n);
  if (p_begin >= n) return;
  const int cl = lane & 15, qd = lane >> 4;

  // page ids and masks, staged once; past the range the last page again, with no valid slot
  const int np = p_end - p_begin;
  {
    const int32_t* trow = table + (size_t)h * max_pages + p_begin;
    const uint16_t* mrow = masks + (size_t)h * max_pages + p_begin;
    for (int i = threadIdx.x; i < np; i += DEC_NT) {
      s_pid[i] = trow[i];
      s_pm[i] = mrow[i];
    }
  }
  // the query rows as B operand: query cl, zero past the group
  bf16x8 qf[KS];
  {
    const uint16_t* row = q + ((size_t)s * Hq + kv * G + min(cl, G - 1)) * D + qd * 8;
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      u32x4 u = *reinterpret_cast<const u32x4*>(row + i * 32);
      if (cl >= G) u = u32x4{0u, 0u, 0u, 0u};
      qf[i] = __builtin_bit_cast(bf16x8, u);
    }
  }
  __syncthreads();

  float m_run, l_run;                       // of query cl, this lane's keys
  f32x4 acc[VE];                            // query 4 qd + r, dim VE cl + e
  // this wave's pairs: pages 2 (wave + DEC_NW j) and the next, j < npair
  const int pairs = (np + 1) >> 1;
  const int npair = wave < pairs ? (pairs - 1 - wave) / DEC_NW + 1 : 0;
  u32x4 kf[2][KS];
  vpiece vf[8];
  auto load_k = [&](int j) {
    const int p0 = 2 * (wave + DEC_NW * min(j, npair - 1));
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const size_t page = (size_t)s_pid[min(p0 + t, np - 1)] * HK_PAGE;
      const uint16_t* src = k_pool + (page + cl) * D + qd * 8;
#pragma unroll
      for (int i = 0; i < KS; ++i) kf[t][i] = *reinterpret_cast<const u32x4*>(src + i * 32);
    }
  };
  auto load_v = [&](int j) {
    const int p0 = 2 * (wave + DEC_NW * min(j, npair - 1));
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const size_t page = (size_t)s_pid[min(p0 + t, np - 1)] * HK_PAGE;
      const uint16_t* src = v_pool + (page + 4 * qd) * D + cl * VE;
#pragma unroll
      for (int i = 0; i < 4; ++i) vf[4 * t + i] = *reinterpret_cast<const vpiece*>(src + i * D);
    }
  };
  // COLD: the walk again, where a sum came out NaN or too large: a new reference with every
  // larger score (no probability above 1), and with `lead` the leading part of P for all three
  auto walk = [&](auto cold, bool lead) {
    constexpr bool COLD = decltype(cold)::value;
    constexpr float SLACK = COLD ? 0.f : DEC_SLACK;
    m_run = -INFINITY;
    l_run = 0.f;
#pragma unroll
    for (int e = 0; e < VE; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (npair > 0) {
      load_k(0);
      load_v(0);
    }
    float sf = 1.f;                           // the sign this pair's products are formed with
    for (int j = 0; j < npair; ++j) {
      const float cs = sf * c2;
      const int p0 = 2 * (wave + DEC_NW * j);
      const uint32_t m32 = (uint32_t)s_pm[p0] | (p0 + 1 < np ? (uint32_t)s_pm[p0 + 1] << 16 : 0u);
      f32x4 z[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 half[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int i = 0; i < KS; ++i)
          half[i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[t][i]), qf[i],
                                                                half[i & 1], 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) z[t][r] = half[0][r] + half[1][r];
      }
      load_k(j + 1);
#pragma unroll
      for (int i = 0; i < KS; ++i) qf[i] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[i]) ^ 0x80008000u);
      if (m32 != 0xffffffffu) {
        const uint32_t mm = m32 >> (4 * qd);            // keys 4 qd + r: bits r and 16 + r
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (!((mm >> (16 * t + r)) & 1u)) z[t][r] = -INFINITY * sf;
      }
      float zx = z[0][0], zn = z[0][0];
#pragma unroll
      for (int k = 1; k < 8; ++k) {
        zx = fmaxf(zx, z[k >> 2][k & 3]);
        zn = fminf(zn, z[k >> 2][k & 3]);
      }
      float zm = (sf > 0.f ? zx : zn) * cs;             // the lane's largest, log2 units
      if (__any(zm > m_run + SLACK)) {
        // a new reference: the pair's maximum of each query (its four lanes l % 16 alike)
        zm = fmaxf(zm, __shfl_xor(zm, 16, 64));
        zm = fmaxf(zm, __shfl_xor(zm, 32, 64));
        const float mn = fmaxf(m_run, ceilf(zm));
        const float alpha = m_run == -INFINITY ? 0.f : fast_exp2(m_run - mn);
        m_run = mn;
        l_run *= alpha;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float ar = __shfl(alpha, 4 * qd + r, 64);
#pragma unroll
          for (int e = 0; e < VE; ++e) acc[e][r] *= ar;
        }
      }
      // probabilities (0 where no key has come yet) and their three bf16 parts, two keys a word
      const float mc = m_run == -INFINITY ? 0.f : m_run;
      uint32_t ph[4], pm[4], pl[4];
      float ps[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t a[2], b[2], c[2];
        ps[w] = 0.f;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int k = 2 * w + u;
          float p = fast_exp2(fmaf(z[k >> 2][k & 3], cs, -mc));
          ps[w] += p;
          p *= sf;
          a[u] = __float_as_uint(p);
          const float r1 = p - __uint_as_float(a[u] & 0xffff0000u);
          b[u] = __float_as_uint(r1);
          c[u] = __float_as_uint(r1 - __uint_as_float(b[u] & 0xffff0000u));
        }
        ph[w] = __builtin_amdgcn_perm(a[1], a[0], 0x07060302u);
        pm[w] = __builtin_amdgcn_perm(b[1], b[0], 0x07060302u);
        pl[w] = __builtin_amdgcn_perm(c[1], c[0], 0x07060302u);
      }
      l_run += (ps[0] + ps[1]) + (ps[2] + ps[3]);
      const bf16x8 fh = __builtin_bit_cast(bf16x8, u32x4{ph[0], ph[1], ph[2], ph[3]});
      const bf16x8 fm = __builtin_bit_cast(bf16x8, u32x4{pm[0], pm[1], pm[2], pm[3]});
      const bf16x8 fl = __builtin_bit_cast(bf16x8, u32x4{pl[0], pl[1], pl[2], pl[3]});
      if (COLD && p0 + 1 >= np)               // the last page repeated: no infinity times its 0
#pragma unroll
        for (int i = 4; i < 8; ++i) vf[i] = vpiece{};
#pragma unroll
      for (int w = 0; w < VW; ++w) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const uint32_t sel = u ? 0x07060302u : 0x05040100u;
          u32x4 b;
#pragma unroll
          for (int i = 0; i < 4; ++i) b[i] = __builtin_amdgcn_perm(vf[2 * i + 1][w], vf[2 * i][w], sel);
          const bf16x8 vb = __builtin_bit_cast(bf16x8, b);
          f32x4 t = {0.f, 0.f, 0.f, 0.f};
          if (!COLD || !lead) {
            t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl, vb, t, 0, 0, 0);
            t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fm, vb, t, 0, 0, 0);
          }
          t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh, vb, t, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[2 * w + u][r] = fmaf(t[r], sf, acc[2 * w + u][r]);
        }
      }
      load_v(j + 1);
      sf = -sf;
    }
  };
  walk(std::false_type{}, false);
  float bad = 0.f;                          // NaN when some sum is NaN or 2^104 or above
#pragma unroll
  for (int e = 0; e < VE; ++e)
#pragma unroll
    for (int r = 0; r < 4; ++r) bad = fmaf(acc[e][r] * 0x1p24f, 0.f, bad);
  auto keep = [&](bool only_nan) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * qd + r < G)
#pragma unroll
        for (int e = 0; e < VE; ++e) {
          float* at = &s_o[wave][4 * qd + r][cl * VE + e];
          if (!only_nan || *at != *at) *at = acc[e][r];
        }
  };
  keep(false);
  if (__any(bad != bad)) {
    // Values near the end of the fp32 range overflow, here or where the states are merged,
    // against a reference that lies below the largest score: the walk is done again with
    // references that no score exceeds.  An infinite value times a part of P that is 0 is NaN
    // where value times P is infinite: sums that are NaN after that walk are taken from a third
    // one with the leading part alone.
    for (int lead = 0; lead < 2; ++lead) {
      if (npair & 1)                        // the queries' sign as at the start
#pragma unroll
        for (int i = 0; i < KS; ++i) qf[i] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[i]) ^ 0x80008000u);
      walk(std::true_type{}, lead);
      keep(lead);
    }
  }
  // the four lanes of a query hold its sum in parts
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (lane < G) {
    s_m[wave][lane] = m_run;
    s_l[wave][lane] = l_run;
  }
  __syncthreads();
  // combine the waves -> one partial state per (head, split, g): [o(D) unnormalised, m, l]
  for (int idx = threadIdx.x; idx < G * D; idx += DEC_NT) {
    const int g = idx / D, d = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < DEC_NW; ++w) M = fmaxf(M, s_m[w][g]);
    float L = 0.f, O = 0.f;
    if (M != -INFINITY)
#pragma unroll
      for (int w = 0; w < DEC_NW; ++w) {
        const float a = fast_exp2(s_m[w][g] - M);
        L += s_l[w][g] * a;
        O += s_o[w][g][d] * a;
      }
    float* dst = part + (((size_t)h * n_split + split) * G + g) * (D + 2);
    dst[d] = O;
    if (d == 0) {
      dst[D] = M;
      dst[D + 1] = L;
    }
  }
}

// NW waves per query head merge its split states (App. F).  Lanes hold two output columns
// each, and a group of D / 2 lanes takes every NG-th split, U of them in flight at once, so
// the chain of dependent loads is n_split / (NG * U) long.  Every wave reads all (m, l) itself
// (64 splits per load) for the running maximum M and the rescaled sum L; a split's own factor
// exp2(m - M) comes from the m loaded beside its outputs.  The first batch of loads -- page
// count, states and outputs -- is issued before the number of splits that held pages is
// known; the states of the others are dropped unread (their memory holds an earlier call's
// values).  Launches of at most 8 splits take one wave per query head, which then has every
// split in flight; more splits take four waves.  Up to 32 splits of more than MRG_MANY query
// heads stay at one: those waves fill the chip, and four times as many only queue and load
// dead splits (1024 heads x 4 x 12 splits 10.2 us with four waves, 6.5 with one, 6.8 with one
// workgroup per KV head; 488 x 4 x 16 6.3, 4.8 and 6.7).  Bound by the latency of two or three
// dependent loads: 16 heads x 7 query heads x 128 splits 45.6 -> 5.5 us against one workgroup
// per KV head with four loads in flight per thread, 16 x 4 x 48 splits 11.3 -> 4.0 us, 512 x 4 x 6
// splits 4.9 -> 3.7 us over a whole decode loop.
constexpr int MRG_NT = 256;
constexpr int MRG_MANY = 1024;               // query heads that fill the chip with one wave each
template <int D, int NW, int U>
__global__ __launch_bounds__(MRG_NT) void decode_merge_kernel(const float* __restrict__ part,
                                                              const int32_t* __restrict__ n_pages_arr,
                                                              int max_pages, int n_split_all, int pps,
                                                              int n_q, int G, int Hq, int Hkv,
                                                              float* __restrict__ o,
                                                              float* __restrict__ lse) {
  constexpr int LPS = D / 2;                  // lanes per split, two columns each
  constexpr int TPQ = 64 * NW;                // threads per query head
  constexpr int NG = TPQ / LPS;               // lane groups
  __shared__ float2 s_o[MRG_NT / TPQ][NG][LPS];
  const int qi = threadIdx.x / TPQ, tq = threadIdx.x % TPQ;
  // past the last query head: the last one again, not stored
  const int q_row = (int)blockIdx.x * (MRG_NT / TPQ) + qi, q_cl = min(q_row, n_q - 1);
  const int h = q_cl / G, g = q_cl % G;
  const int s = h / Hkv, kv = h % Hkv;
  const int lane = threadIdx.x & 63, grp = tq / LPS, col = tq % LPS;
  const size_t stride = (size_t)G * (D + 2);
  const float* base = part + (size_t)h * n_split_all * stride + (size_t)g * (D + 2);
  const int n = min(n_pages_arr[h], max_pages);
  // (m, l) of the splits lane and lane + 64; outputs and m of the splits grp + NG * (j0 + u),
  // clamped to the launch's last split
  auto load_ml = [&](int i) {
    return i < n_split_all ? *reinterpret_cast<const float2*>(base + i * stride + D) : make_float2(-INFINITY, 0.f);
  };
  float2 ml0 = load_ml(lane), ml1 = load_ml(lane + 64);
  float2 ov[U];
  float mv[U];
  auto load_o = [&](int j0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(grp + NG * (j0 + u), n_split_all - 1);
      const float* p = base + i * stride;
      ov[u] = *reinterpret_cast<const float2*>(p + 2 * col);
      mv[u] = p[D];
    }
  };
  load_o(0);
  const int share = decode_share(n, n_split_all, pps);
  const int n_split = n > 0 ? min(n_split_all, (n + share - 1) / share) : 0;
  if (lane >= n_split) ml0 = make_float2(-INFINITY, 0.f);
  if (lane + 64 >= n_split) ml1 = make_float2(-INFINITY, 0.f);
  float M = fmaxf(ml0.x, ml1.x);
  for (int i = lane + 128; i < n_split; i += 64) M = fmaxf(M, base[i * stride + D]);
  M = wave_max(M);
  float L = 0.f;
  float2 acc = make_float2(0.f, 0.f);
  if (M != -INFINITY) {                       // the same in every wave
    if (lane < n_split) L += ml0.y * exp2f(ml0.x - M);
    if (lane + 64 < n_split) L += ml1.y * exp2f(ml1.x - M);
    for (int i = lane + 128; i < n_split; i += 64) {
      const float2 ml = *reinterpret_cast<const float2*>(base + i * stride + D);
      L += ml.y * exp2f(ml.x - M);
    }
    L = wave_sum(L);
    for (int j0 = 0;;) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (grp + NG * (j0 + u) < n_split) {
          const float a = exp2f(mv[u] - M);
          acc.x = fmaf(ov[u].x, a, acc.x);
          acc.y = fmaf(ov[u].y, a, acc.y);
        }
      j0 += U;
      if (NG * j0 >= n_split) break;
      load_o(j0);
    }
  }
  s_o[qi][grp][col] = acc;
  __syncthreads();
  const size_t row = (size_t)s * Hq + kv * G + g;
  if (tq < LPS && q_row < n_q) {
    float2 t = s_o[qi][0][col];
#pragma unroll
    for (int q = 1; q < NG; ++q) {
      t.x += s_o[qi][q][col].x;
      t.y += s_o[qi][q][col].y;
    }
    o[row * D + 2 * col] = L > 0.f ? t.x / L : 0.f;        // (o need not be 8-byte aligned)
    o[row * D + 2 * col + 1] = L > 0.f ? t.y / L : 0.f;
  }
  if (tq == 0 && q_row < n_q) lse[row] = (L > 0.f) ? (M + __log2f(L)) * kLn2 : -INFINITY;
}

// ------------------------------------------------------------------ a6: append
// Two launches.  Count: one wave per 64 heads records how many of its heads need a fresh
// page (row empty, or newest page full) and whether any such row is already at max_pages,
// and block 0 snapshots the free-list top.  Write: every workgroup re-derives its heads'
// needs, takes the exclusive prefix over the preceding workgroups' counts (head order, so
// the pops are the same as a sequential scan), decides success from the global totals,
// and writes its heads.  Only block 0 updates free_top; every block reads the snapshot.
// Workspace (int32): [0] top snapshot, [1, 1+nblk) counts, [1+nblk, 1+2*nblk) full flags.
constexpr int AP_HPB = 64;     // heads per workgroup
constexpr int AP_NT = 256;

__device__ inline void append_need(int h, int n_heads, const int32_t* n_pages, const uint16_t* masks,
                                   int max_pages, int& n, uint32_t& m, int& need, int& full) {
  n = 0;
  m = 0;
  need = 0;
  full = 0;
  if (h >= n_heads) return;
  n = n_pages[h];
  m = n > 0 ? masks[(size_t)h * max_pages + n - 1] : 0xffffu;
  if ((m & 0x8000u) || n == 0) {
    need = 1;
    full = n >= max_pages;
  }
}

__global__ __launch_bounds__(64) void append_count_kernel(int n_heads, const int32_t* __restrict__ n_pages,
                                                          const uint16_t* __restrict__ masks, int max_pages,
                                                          const int32_t* __restrict__ free_top,
                                                          int32_t* __restrict__ ws) {
  const int nblk = gridDim.x;
  int n, need, full;
  uint32_t m;
  append_need(blockIdx.x * AP_HPB + threadIdx.x, n_heads, n_pages, masks, max_pages, n, m, need, full);
  need = wave_sum(need);
  full = __any(full) ? 1 : 0;
  if (threadIdx.x == 0) {
    ws[1 + blockIdx.x] = need;
    ws[1 + nblk + blockIdx.x] = full;
    if (blockIdx.x == 0) ws[0] = *free_top;
  }
}

template <int ROW_BYTES>
__global__ __launch_bounds__(AP_NT) void append_write_kernel(
    int n_heads, char* __restrict__ k_pool, char* __restrict__ v_pool, int32_t* __restrict__ table,
    uint16_t* __restrict__ masks, int32_t* __restrict__ n_pages, int max_pages,
    const char* __restrict__ k_new, const char* __restrict__ v_new, const int32_t* __restrict__ free_ids,
    int32_t* __restrict__ free_top, int32_t* __restrict__ status, const int32_t* __restrict__ ws) {
  constexpr int CH = ROW_BYTES / 16;
  __shared__ int s_red[3][AP_NT / 64];
  __shared__ int64_t s_dst[AP_HPB];
  const int nblk = gridDim.x, blk = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // global totals and this block's offset, from the counts of the first launch
  int before = 0, total = 0, anyfull = 0;
  for (int b = threadIdx.x; b < nblk; b += AP_NT) {
    const int c = ws[1 + b];
    total += c;
    if (b < blk) before += c;
    anyfull |= ws[1 + nblk + b];
  }
  before = wave_sum(before);
  total = wave_sum(total);
  anyfull = __any(anyfull) ? 1 : 0;
  if (lane == 0) {
    s_red[0][wave] = before;
    s_red[1][wave] = total;
    s_red[2][wave] = anyfull;
  }
  __syncthreads();
  before = total = anyfull = 0;
#pragma unroll
  for (int w = 0; w < AP_NT / 64; ++w) {
    before += s_red[0][w];
    total += s_red[1][w];
    anyfull |= s_red[2][w];
  }
  const int top = ws[0];
  const bool ok = !anyfull && total <= top;
  if (blk == 0 && threadIdx.x == 0) {
    if (ok) *free_top = top - total;
    else if (status) atomicOr(status, HK_FLAG_NOSPACE);
  }
  if (!ok) return;
  if (wave == 0) {
    const int h = blk * AP_HPB + lane;
    int n, need, full;
    uint32_t m;
    append_need(h, n_heads, n_pages, masks, max_pages, n, m, need, full);
    int x = need;   // inclusive scan over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    int64_t dst = -1;
    if (h < n_heads) {
      int page, slot;
      if (need) {
        page = free_ids[top - total + before + x - 1];
        table[(size_t)h * max_pages + n] = page;
        masks[(size_t)h * max_pages + n] = 1;
        n_pages[h] = n + 1;
        slot = 0;
      } else {
        page = table[(size_t)h * max_pages + n - 1];
        slot = 32 - __clz(m);               // one past the highest valid slot
        masks[(size_t)h * max_pages + n - 1] = (uint16_t)(m | (1u << slot));
      }
      dst = ((int64_t)page * HK_PAGE + slot) * ROW_BYTES;
    }
    s_dst[lane] = dst;
  }
  __syncthreads();
  // rows of the workgroup's heads: K then V, 16-byte chunks, consecutive threads on one row
  const int h0 = blk * AP_HPB;
  for (int i = threadIdx.x; i < 2 * AP_HPB * CH; i += AP_NT) {
    const int kv = i / (AP_HPB * CH), r = i % (AP_HPB * CH);
    const int hl = r / CH, ch = r % CH;
    const int64_t dst = s_dst[hl];
    if (dst < 0) continue;
    const size_t src = (size_t)(h0 + hl) * ROW_BYTES + ch * 16;
    const uint4 u = *reinterpret_cast<const uint4*>((kv ? v_new : k_new) + src);
    *reinterpret_cast<uint4*>((kv ? v_pool : k_pool) + dst + ch * 16) = u;
  }
}

template <int D>
static void launch_split(int G, dim3 grid, hipStream_t st, const void* q, const hk_paged_kv* kv, int Hq,
                         int Hkv, float c2, float* part, int n_split, int pps, uint32_t heads_first) {
  hipLaunchKernelGGL(decode_split_kernel<D>, grid, dim3(DEC_NT), 0, st, static_cast<const uint16_t*>(q),
                     static_cast<const uint16_t*>(kv->k_pool), static_cast<const uint16_t*>(kv->v_pool),
                     kv->page_table, kv->page_mask, kv->n_pages, G, Hq, Hkv, kv->max_pages, c2, part,
                     n_split, pps, heads_first);
}

template <int D, int G>
static void launch_split_f32(dim3 grid, hipStream_t st, const void* q, const hk_paged_kv* kv, int Hq,
                             int Hkv, float c2, float* part, int n_split, int pps) {
  hipLaunchKernelGGL((decode_split_f32_kernel<D, G>), grid, dim3(DEC_NT), 0, st,
                     static_cast<const float*>(q), static_cast<const float*>(kv->k_pool),
                     static_cast<const float*>(kv->v_pool), kv->page_table, kv->page_mask, kv->n_pages,
                     Hq, Hkv, kv->max_pages, c2, part, n_split, pps);
}

template <int D>
static void launch_split_f32_g(int G, dim3 grid, hipStream_t st, const void* q, const hk_paged_kv* kv,
                               int Hq, int Hkv, float c2, float* part, int n_split, int pps) {
  switch (G) {
    case 1: launch_split_f32<D, 1>(grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps); break;
    case 2: launch_split_f32<D, 2>(grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps); break;
    case 4: launch_split_f32<D, 4>(grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps); break;
    case 7: launch_split_f32<D, 7>(grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps); break;
    default: launch_split_f32<D, 8>(grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps); break;
  }
}

}  // namespace hk

using namespace hk;

bool hk_decode_supports_group(int G) { return G == 1 || G == 2 || G == 4 || G == 7 || G == 8; }

size_t hk_decode_ws(int NS, int Hq, int Hkv, int D, int max_pages) {
  const int G = Hq / Hkv, n_split = (max_pages + DEC_PPS_MIN - 1) / DEC_PPS_MIN;
  return (size_t)NS * Hkv * n_split * G * (D + 2) * sizeof(float);
}

void hk_decode_split_plan(int n_heads, int max_pages, int* pps_out, int* n_split_out) {
  // pages per split: the most (DEC_PPS) that still gives the launch DEC_TARGET_WG
  // workgroups, down to DEC_PPS_MIN -- few heads get short splits, so no wave walks a
  // long serial chain of pages
  int pps = DEC_PPS;
  while (pps > DEC_PPS_MIN && (long long)n_heads * ((max_pages + pps - 1) / pps) < DEC_TARGET_WG)
    pps >>= 1;
  *pps_out = pps;
  *n_split_out = (max_pages + pps - 1) / pps;
}

hipError_t hk_launch_decode(int NS, int Hq, int Hkv, int D, const void* q, const hk_paged_kv* kv,
                            float sm_scale, float* o, float* lse, void* ws, hipStream_t st,
                            bool timed) {
  const int G = Hq / Hkv, n_heads = NS * Hkv;
  int pps, n_split;
  hk_decode_split_plan(n_heads, kv->max_pages, &pps, &n_split);
  const float c2 = sm_scale * kLog2e;
  float* part = static_cast<float*>(ws);
  const bool bf = kv->dtype == HK_BF16;
  // One or two query heads of a bf16 cache: the launch runs over the heads first, so that the
  // splits past the rows' ends come last.  With a head's splits in turn they lie between the
  // others, and as workgroups go to the eight dies and their CUs in turn, the first 3 splits of
  // 16 all fall to three dies.  There the matrix-core kernel was slower than the VALU form had
  // been: 512 heads of 641 tokens in a 32768-token table, G 1, 70 us (VALU form), 107, heads first
  // 32; G 2 87, 109, 33; 64 heads of 640 in 12288 at G 1 16.5, 21.9, 11.2.  From 4 query heads on it
  // was faster in that order too, and where most splits hold pages that order is better by up
  // to 4% (16 heads x 7 x 23k to 33k tokens 55.6 us, heads first 57.1).  The heads are turned
  // by the split, or a head's splits would all meet on one die.
  const bool by_heads = bf && G <= 2 && n_split <= 65535;
  const uint32_t heads_first = by_heads ? turn_magic(n_heads) : 0u;
  const dim3 grid(by_heads ? n_heads : n_split, by_heads ? n_split : n_heads);
  if (!hk_decode_supports_group(G)) return hipErrorInvalidValue;
  {
    TimedLaunch t(timed ? HK_TK_DECODE_SPLIT : -1, st);
    if (bf && D == 128) launch_split<128>(G, grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps, heads_first);
    else if (bf) launch_split<64>(G, grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps, heads_first);
    else if (D == 128) launch_split_f32_g<128>(G, grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps);
    else launch_split_f32_g<64>(G, grid, st, q, kv, Hq, Hkv, c2, part, n_split, pps);
  }
  TimedLaunch t(timed ? HK_TK_DECODE_MERGE : -1, st);
  const int n_q = n_heads * G;
#define HK_MERGE(D_, NW_, U_)                                                                      \
  hipLaunchKernelGGL((decode_merge_kernel<D_, NW_, U_>), dim3((n_q * NW_ + 3) / 4), dim3(MRG_NT), 0, \
                     st, part, kv->n_pages, kv->max_pages, n_split, pps, n_q, G, Hq, Hkv, o, lse)
  const bool one_wave = n_split <= 8 || (n_q > MRG_MANY && n_split <= 32);
  if (D == 128) {
    if (one_wave) HK_MERGE(128, 1, 8);
    else HK_MERGE(128, 4, 8);
  } else {
    if (n_split <= 8) HK_MERGE(64, 1, 4);
    else if (one_wave) HK_MERGE(64, 1, 8);
    else HK_MERGE(64, 4, 8);
  }
#undef HK_MERGE
  return hipGetLastError();
}

// ------------------------------------------------------------------ decode without allocation
// The split partial states of hk_decode_attn_noalloc live in this file-scope device array
// instead of a caller workspace: one copy per GPU the library runs on, held until the
// process ends.  Host code never uses the array's name as an address: its device address is
// looked up once per device (with that device current) and kept here.
static __device__ __align__(256) char scratch[HK_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t hk_noalloc_scratch(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

size_t hk_decode_noalloc_bytes(int NS, int Hq, int Hkv, int D, int max_pages) {
  int pps, n_split;
  hk_decode_split_plan(NS * Hkv, max_pages, &pps, &n_split);
  return (size_t)NS * Hkv * n_split * (Hq / Hkv) * (D + 2) * sizeof(float);
}

size_t hk_append_ws(int NS, int Hkv) {
  const int nblk = (NS * Hkv + AP_HPB - 1) / AP_HPB;
  return (size_t)(1 + 2 * nblk) * sizeof(int32_t);
}

hipError_t hk_launch_append(int NS, int Hkv, int D, const hk_paged_kv* kv, const void* k_new,
                            const void* v_new, const hk_allocator* alloc, int32_t* status, void* ws,
                            hipStream_t st) {
  const int n_heads = NS * Hkv, nblk = (n_heads + AP_HPB - 1) / AP_HPB;
  const int row_bytes = D * (kv->dtype == HK_BF16 ? 2 : 4);
  char* kp = static_cast<char*>(kv->k_pool);
  char* vp = static_cast<char*>(kv->v_pool);
  const char* kn = static_cast<const char*>(k_new);
  const char* vn = static_cast<const char*>(v_new);
  int32_t* w = static_cast<int32_t*>(ws);
  TimedLaunch t(HK_TK_APPEND, st);
  hipLaunchKernelGGL(append_count_kernel, dim3(nblk), dim3(64), 0, st, n_heads, kv->n_pages,
                     kv->page_mask, kv->max_pages, alloc->free_top, w);
#define HK_APPEND_WRITE(RB)                                                                       \
  hipLaunchKernelGGL((append_write_kernel<RB>), dim3(nblk), dim3(AP_NT), 0, st, n_heads, kp, vp, \
                     kv->page_table, kv->page_mask, kv->n_pages, kv->max_pages, kn, vn,           \
                     alloc->free_ids, alloc->free_top, status, w)
  switch (row_bytes) {
    case 128: HK_APPEND_WRITE(128); break;
    case 256: HK_APPEND_WRITE(256); break;
    default: HK_APPEND_WRITE(512); break;
  }
#undef HK_APPEND_WRITE
  return hipGetLastError();
}
