// Chunked causal prefill (Sec. 2: the decode formulation carries over to
// prefill and training). The T positions of a chunk are decoded together,
// each query exactly as a decode step at its own position would be: its own
// block selection, the statistics of the units it shares with the chunk
// taken over the tokens up to its position, and S_bar over its prefix.
//
//   prefill_partial_kernel  log masses of the units in progress at each
//                           position (their running mean and M2)
//   (append_blocks_kernel)  the chunk's K/V rows and unit statistics
//   (append_state_mfma_kernel, block-aligned)  phi(K)^T V of every block the
//                           chunk touches
//   prefill_prefix_kernel   S_bar before each of those blocks, as matrix-core
//                           operands; S_bar and z_bar past the chunk
//   prefill_score_kernel    every query's block scores on the matrix cores;
//                           each statistics tile is loaded once
//   prefill_select_kernel   every query's top-k; prefill_rescore_kernel and a
//                           second selection for the queries whose cutoff the
//                           rounding of the scores could move (short chunks are
//                           scored by prefill_rescore_kernel alone)
//   prefill_group_kernel    the fused exact + linear pass for groups of
//                           consecutive queries over the union of their
//                           selections
//   prefill_merge_kernel    (only where a group's blocks are split over
//                           several workgroups) residual, RMSNorm, output
//
// Query i of a chunk starting at L0 (the sequence length before it) sees
// L_i = L0 + min(i + 1, nv) tokens, nv being the chunk positions that fit
// below the capacity (a query past the capacity decodes over the full cache,
// as a decode step at capacity does).
#include "spla_kernels.h"
#include "spla_score.h"
#include "spla_select.h"
#include "spla_sparse.h"

namespace spla {

constexpr int kPrefSelThreads = 1024;  // threads of a selection workgroup

__device__ __forceinline__ void chunk_bounds(const Dims& m, const int32_t* __restrict__ seq_lens,
                                             int b, int T, int* L0, int* nv) {
  const int l0 = min(max(seq_lens[b], 0), m.cap);
  *L0 = l0;
  *nv = min(m.cap - l0, T);
}

// first unit holding token L0 (u us + ul > L0)
__device__ __forceinline__ int first_touched_unit(const Dims& m, int L0) {
  return L0 >= m.ul ? (L0 - m.ul) / m.us + 1 : 0;
}

constexpr float kLn2f32 = 0.69314718055994531f;

// The queries whose selection is taken again (PrefillWs::near): how many of each
// (sequence, KV head), the largest count, their positions.
struct NearLists {
  int32_t *count, *longest, *list;
};
SPLA_HD NearLists near_lists(const Dims& m, int32_t* near) {
  return {near, near + m.bh, near + m.bh + 1};
}

// ln n + ln(1 + x) as the decode's scoring takes them (hardware log2)
__device__ __forceinline__ double log_mass(double mean_term, int n, float x, int first_order) {
  double ell = mean_term + (double)(__builtin_amdgcn_logf((float)n) * kLn2f32);
  if (!first_order) ell += (double)(__builtin_amdgcn_logf(1.0f + x) * kLn2f32);
  return ell;
}

// exp(ell - tmx) as the decode's scoring takes it; 0 for a unit that is not there
__device__ __forceinline__ float exp_mass(double ell, double tmx) {
  const double t = (ell - tmx) * 1.4426950408889634;
  const float th = (float)t, tl = (float)(t - (double)th);
  const float eh = __builtin_amdgcn_exp2f(th);
  return ell > -INFINITY ? fmaf(eh, tl * kLn2f32, eh) : 0.f;
}

// --------------------------------------------------- units in progress
// Unit first + ur of (sequence, KV head) bh, for every chunk position i whose
// token lies in it: the unit's mean and M2 over its tokens up to position i
// (running sums of k and k^2 in fp64, rounded to fp32 as the stored
// statistics are), and from them the log block mass of every query head
// (Eqs. 8 and 10), to ell_part[bh][i][w][head], w counting the units that
// hold the token from the last one back. Sixteen positions at a time: thread
// j < d forms the statistics of coordinate j, then d / 8 lanes per position
// take the dot products with the decode's arithmetic (eight coordinates in
// fp32, those partial sums in fp64). Runs before the rows are appended (it
// reads the statistics the cache held before the chunk).
template <int D>
__global__ __launch_bounds__(256) void prefill_partial_kernel(
    Dims m, int T_, int W, const float* __restrict__ stats, const int32_t* __restrict__ seq_lens,
    const bf16_t* __restrict__ k_new, const bf16_t* __restrict__ q, double s, int first_order,
    double* __restrict__ ell_part) {
  constexpr int NP = 16, LP = D / 8;  // positions per pass, lanes per position
  __shared__ __align__(16) float s_mean[NP][D + 4], s_m2[NP][D + 4];
  const int bh = blockIdx.y, b = bh / m.hkv, h = bh % m.hkv, G = m.group;
  int L0, nv;
  chunk_bounds(m, seq_lens, b, T_, &L0, &nv);
  const int u = first_touched_unit(m, L0) + (int)blockIdx.x;
  const int64_t u0 = (int64_t)u * m.us;
  const int lo = (int)max(u0, (int64_t)L0), hi = (int)min(u0 + m.ul, (int64_t)L0 + nv);
  if (hi <= lo || (hi + m.B - 1) / m.B <= m.k) return;  // nothing here, or every block selected
  const int tid = threadIdx.x, j = tid % D;
  double s1 = 0.0, s2 = 0.0;
  if (u0 < L0) {  // the unit's tokens before the chunk
    const double na = (double)(L0 - u0);
    const double mean = stats[stats_off4(m, bh, u, 0, j / 4) + (j & 3)];
    const double m2 = stats[stats_off4(m, bh, u, 1, j / 4) + (j & 3)];
    s1 = na * mean;
    s2 = m2 + na * mean * mean;
  }
  for (int t0 = lo; t0 < hi; t0 += NP) {
    const int nt = min(NP, hi - t0);
    if (tid < D) {
      float x[NP];
#pragma unroll
      for (int e = 0; e < NP; ++e)
        x[e] = Elem<bf16_t>::load(k_new,
                                  ((int64_t)(min(t0 + e, hi - 1) - L0) * m.bh + bh) * D + j);
#pragma unroll
      for (int e = 0; e < NP; ++e) {
        s1 += (double)x[e];
        s2 += (double)x[e] * (double)x[e];
        const double mean = s1 / (double)(t0 + e + 1 - u0);
        s_mean[e][j] = (float)mean;  // entries past nt are not used (and end the unit)
        s_m2[e][j] = (float)(s2 - mean * s1);
      }
    }
    __syncthreads();
    const int p = tid / LP, c0 = 8 * (tid % LP), pe = min(p, nt - 1);
    const int i = t0 + pe - L0;  // position within the chunk
    const int n = t0 + pe + 1 - (int)u0;
    if (p < NP) {
      for (int g = 0; g < G; ++g) {
        const bf16_t* qr = q + (((int64_t)i * m.batch + b) * m.hq + h * G + g) * D + c0;
        float pm = 0.f, pv = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double x = (double)bf16_to_f32(qr[e].bits);
          pm = fmaf((float)(s * x), s_mean[pe][c0 + e], pm);
          pv = fmaf((float)(0.5 * s * s * x * x), s_m2[pe][c0 + e], pv);
        }
        double dm = (double)pm, dv = (double)pv;
#pragma unroll
        for (int sft = 1; sft < LP; sft *= 2) {
          dm += __shfl_xor(dm, sft, LP);
          dv += __shfl_xor(dv, sft, LP);
        }
        if (tid % LP == 0 && p < nt) {
          const int w = (t0 + p) / m.us - u;  // 0 .. W - 1
          ell_part[(((int64_t)bh * T_ + i) * W + w) * G + g] =
              log_mass(dm, n, (float)dv * __builtin_amdgcn_rcpf((float)n), first_order);
        }
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------- prefix
// From the block partials P_x = sum phi(k)^T v (x = 0 the block of position
// L0) of one (sequence, KV head): S_bar before block x, S_x = S + P_0 + ... +
// P_{x-1} (summed in fp64 in block order, rounded to fp32), written as the
// A operand of S_x^T (tile t, k-step ks: lane holds coordinate 16 t + lane %
// 16, rows 32 ks + 8 (lane / 16) .. + 7 of S_x) in bf16 hi + lo, z_x in fp32;
// then S_bar and z_bar past the chunk. One thread per eight rows of one
// column; lin: whether any query needs S_x (else only the state moves on).
template <int D>
__global__ __launch_bounds__(256) void prefill_prefix_kernel(
    Dims m, int T_, int n_blk, int lin, const int32_t* __restrict__ seq_lens,
    const float* __restrict__ part_s, const float* __restrict__ part_z, float* __restrict__ S,
    float* __restrict__ zbar, uint4* __restrict__ s_hi, uint4* __restrict__ s_lo,
    float* __restrict__ z_pre, int32_t* __restrict__ near) {
  constexpr int KS = D / 32, PER = D * D / 8;  // operand pieces per block
  const int bh = blockIdx.y;
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // for the selection
    const NearLists nl = near_lists(m, near);
    nl.count[bh] = 0;
    if (bh == 0) *nl.longest = 0;
  }
  int L0, nv;
  chunk_bounds(m, seq_lens, bh / m.hkv, T_, &L0, &nv);
  if (nv <= 0 && !lin) return;
  const int nx = nv > 0 ? (L0 + nv - 1) / m.B - L0 / m.B + 1 : 0;  // blocks the chunk touches
  const int pc = (int)blockIdx.x * 256 + (int)threadIdx.x;
  const int lane = pc & 63, ks = (pc >> 6) % KS, t = (pc >> 6) / KS;
  const int64_t e0 = (int64_t)(32 * ks + 8 * (lane >> 4)) * D + 16 * t + (lane & 15);
  float* Sb = S + (int64_t)bh * D * D + e0;
  const float* P = part_s + (int64_t)bh * n_blk * D * D + e0;
  double acc[8];
  float nx8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = (double)Sb[(int64_t)e * D];
#pragma unroll
  for (int e = 0; e < 8; ++e) nx8[e] = nx > 0 ? P[(int64_t)e * D] : 0.f;
  for (int x = 0; x < max(nx, 1); ++x) {
    float cur[8], f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cur[e] = nx8[e];
    if (x + 1 < nx) {
#pragma unroll
      for (int e = 0; e < 8; ++e) nx8[e] = P[((int64_t)(x + 1) * D + e) * D];
    }
    if (lin) {
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = (float)acc[e];
      bf16x8 hi, lo;
      split_bf16x8(f, hi, lo);
      s_hi[((int64_t)bh * n_blk + x) * PER + pc] = __builtin_bit_cast(uint4, hi);
      s_lo[((int64_t)bh * n_blk + x) * PER + pc] = __builtin_bit_cast(uint4, lo);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += (double)cur[e];
  }
  if (nx > 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) Sb[(int64_t)e * D] = (float)acc[e];
  }
  if (pc < D) {
    double z = (double)zbar[(int64_t)bh * D + pc];
    for (int x = 0; x < max(nx, 1); ++x) {
      z_pre[((int64_t)bh * n_blk + x) * D + pc] = (float)z;
      z += nx > 0 ? (double)part_z[((int64_t)bh * n_blk + x) * D + pc] : 0.0;
    }
    if (nx > 0) zbar[(int64_t)bh * D + pc] = (float)z;
  }
}

// ------------------------------------------------------------- scoring
// x = a + b + c as bf16 pieces (24 mantissa bits: an fp32 value exactly, away
// from the ends of the exponent range).
__device__ __forceinline__ void split3_bf16x8(const float (&x)[8], bf16x8& a, bf16x8& b,
                                              bf16x8& c) {
  float r[8];
  uint32_t hp[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const uint32_t u = __builtin_bit_cast(
        uint32_t, __builtin_convertvector(f32x2{x[2 * p], x[2 * p + 1]}, bf16x2));
    hp[p] = u;
    r[2 * p] = x[2 * p] - __uint_as_float(u << 16);
    r[2 * p + 1] = x[2 * p + 1] - __uint_as_float(u & 0xFFFF0000u);
  }
  a = __builtin_bit_cast(bf16x8, make_uint4(hp[0], hp[1], hp[2], hp[3]));
  split_bf16x8(r, b, c);
}

// One workgroup per (statistics tile of 64 units, sequence x KV head, share
// of the queries), wavefront w taking units 16 w .. 16 w + 15 as the rows of
// its matrix-core tiles. The tile's statistics are loaded once and kept as
// bf16 operands in three pieces (exact fp32 values); the columns are the
// chunk's query rows r = i G + g (position i, head g), 64 at a time, staged
// in LDS as q (exact in bf16) and q^2 in two pieces (exact). Per 32
// coordinates the products of q . mu and q^2 . M2 accumulate in fp32 from the
// small pieces to the large; the four partial sums of q . mu are added in
// fp64. The log masses carry about as much rounding as the decode's but not
// the same, which the selection makes up for where it matters (tie_span).
// Units in progress at a query's position take their log mass from ell_part.
// Results as the decode's scoring leaves them: exp(ell - tile max) per query
// row and unit, (max, sum) per row and tile.
// On the vector unit the products alone took about 570 instructions per query
// and wavefront; on v_mfma_f32_16x16x4_f32 (the decode's fp32 sums bit for
// bit) a chunk of 256 positions at 128K tokens and 4 x 8 units took 645 us,
// matrix and vector cycles (the conversions of sixteen fp32 partials) adding
// up rather than overlapping. 32 positions there (8 units): 126.6 us on the
// vector unit, 50.1 us now.
template <int D>
struct PrefScoreSmem {
  uint4 q[4][D / 32][64], q2h[4][D / 32][64], q2l[4][D / 32][64];  // per column tile
  double mx[4][64], sum[4][64];  // per wavefront and column
};

template <int D>
__global__ __launch_bounds__(256, 2) void prefill_score_kernel(
    Dims m, int T_, int W, const float* __restrict__ stats, const int32_t* __restrict__ seq_lens,
    const bf16_t* __restrict__ q, double s, int first_order, const double* __restrict__ ell_part,
    float* __restrict__ e_vals, double* __restrict__ tile_part, float2* __restrict__ unit_max,
    float* __restrict__ q_norm2) {
  constexpr int KS = D / 32;
  __shared__ PrefScoreSmem<D> sm;
  const int tile = blockIdx.x, bh = blockIdx.z, b = bh / m.hkv, h = bh % m.hkv;
  const int G = m.group, R = T_ * G;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  int L0, nv;
  chunk_bounds(m, seq_lens, b, T_, &L0, &nv);
  const int Lend = L0 + nv;
  // a tile past every query's tokens, or a chunk whose queries all select
  // every block: nothing reads the scores
  if (tile * kTileBlocks * m.us >= Lend || (Lend + m.B - 1) / m.B <= m.k) return;
  bf16x8 mu[3][KS], vr[3][KS];
  {
    const int64_t blk = (int64_t)tile * kTileBlocks + 16 * w + li;
    f32x4 x[KS][2], y[KS][2];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int j4 = 8 * ks + 2 * lg + u;
        x[ks][u] = *reinterpret_cast<const f32x4*>(stats + stats_off4(m, bh, blk, 0, j4));
        y[ks][u] = *reinterpret_cast<const f32x4*>(
            stats + stats_off4(m, bh, blk, first_order ? 0 : 1, j4));
      }
    if (blockIdx.y == 0) {  // for tie_span; a unit that is not finite counts as infinite
      float n2 = 0.f, v = 0.f;
      bool fine = true;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          n2 = fmaf(x[ks][e >> 2][e & 3], x[ks][e >> 2][e & 3], n2);
          const float y1 = first_order ? 0.f : y[ks][e >> 2][e & 3];
          v = fmaxf(v, y1);
          fine = fine & (y1 < INFINITY);
        }
      n2 += xor16(n2);
      n2 += xor32(n2);
      v *= 1.0f / (float)m.us;  // a whole unit has us tokens at least
      const bool there = blk * m.us < Lend;
      n2 = there ? (n2 < INFINITY ? n2 : INFINITY) : 0.f;
      v = there ? (fine ? v : INFINITY) : 0.f;
      n2 = wave_max(n2);
      v = wave_max(v);
      if (lane == 0) unit_max[((int64_t)bh * m.n_tiles + tile) * 4 + w] = make_float2(n2, v);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      float f[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = x[ks][e >> 2][e & 3];
      split3_bf16x8(f, mu[0][ks], mu[1][ks], mu[2][ks]);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = y[ks][e >> 2][e & 3];
      split3_bf16x8(f, vr[0][ks], vr[1][ks], vr[2][ks]);
    }
  }
  const int nbp = m.n_tiles * kTileBlocks;
  const int u_lane = tile * kTileBlocks + 16 * w + 4 * lg;  // this lane's first result row
  // whether every query sees every unit of the tile whole: the last unit ends
  // within the tokens before the chunk
  const bool inner = (int64_t)((tile + 1) * kTileBlocks - 1) * m.us + m.ul <= L0;  // uniform
  const float half_s2 = (float)(0.5 * s * s);
  const float half_s2_ul = half_s2 * __builtin_amdgcn_rcpf((float)m.ul);
  const int n_cg = (R + 63) / 64;
  for (int cg = blockIdx.y; cg < n_cg; cg += gridDim.y) {
    const int r_hi = min(R, 64 * cg + 64) - 1;
    if ((L0 + min(r_hi / G + 1, nv) + m.B - 1) / m.B <= m.k) continue;  // uniform
    {  // stage column tile w
      const int r = 64 * cg + 16 * w + li;
      const bool ok = r < R;
      const int i = ok ? r / G : 0, g = ok ? r % G : 0;
      const bf16_t* qr = q + (((int64_t)i * m.batch + b) * m.hq + h * G + g) * D + 8 * lg;
      uint4 raw[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) raw[ks] = *reinterpret_cast<const uint4*>(qr + 32 * ks);
      float n2 = 0.f;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 v = __builtin_bit_cast(bf16x8, raw[ks]);
        float f[8];
        bf16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          f[e] = (float)v[e] * (float)v[e];
          n2 += f[e];
        }
        split_bf16x8(f, hi, lo);
        sm.q[w][ks][lane] = raw[ks];
        sm.q2h[w][ks][lane] = __builtin_bit_cast(uint4, hi);
        sm.q2l[w][ks][lane] = __builtin_bit_cast(uint4, lo);
      }
      if (tile == 0) {  // uniform
        n2 += xor16(n2);
        n2 += xor32(n2);
        if (ok && lg == 0) q_norm2[(int64_t)bh * R + r] = n2;
      }
    }
    __syncthreads();
    double ell[4][4];  // column tile, result row
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      floatx4 am[KS], av[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 qv = __builtin_bit_cast(bf16x8, sm.q[ct][ks][lane]);
        const bf16x8 qh = __builtin_bit_cast(bf16x8, sm.q2h[ct][ks][lane]);
        const bf16x8 ql = __builtin_bit_cast(bf16x8, sm.q2l[ct][ks][lane]);
        am[ks] = av[ks] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 2; c >= 0; --c)
          am[ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(mu[c][ks], qv, am[ks], 0, 0, 0);
        av[ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vr[2][ks], qh, av[ks], 0, 0, 0);
        av[ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vr[1][ks], ql, av[ks], 0, 0, 0);
        av[ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vr[1][ks], qh, av[ks], 0, 0, 0);
        av[ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vr[0][ks], ql, av[ks], 0, 0, 0);
        av[ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vr[0][ks], qh, av[ks], 0, 0, 0);
      }
      double dm[4];
      float dv[4];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        dm[rr] = (double)am[0][rr];
        dv[rr] = av[0][rr];
#pragma unroll
        for (int ks = 1; ks < KS; ++ks) {
          dm[rr] += (double)am[ks][rr];
          dv[rr] += av[ks][rr];
        }
        dm[rr] *= s;
      }
      if (inner) {
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
          ell[ct][rr] = log_mass(dm[rr], m.ul, dv[rr] * half_s2_ul, first_order);
      } else {
        const int r = min(64 * cg + 16 * ct + li, R - 1), i = r / G;
        const int L = L0 + min(i + 1, nv), nu = (L + m.us - 1) / m.us;
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int u = u_lane + rr;
          const int n = min(m.ul, max(L - u * m.us, 1));
          double x = log_mass(dm[rr], n, dv[rr] * half_s2 * __builtin_amdgcn_rcpf((float)n),
                              first_order);
          const int wu = (L0 + i) / m.us - u;
          if (i < nv && wu >= 0 && wu < W)
            x = ell_part[(((int64_t)bh * T_ + i) * W + wu) * G + (r - i * G)];
          ell[ct][rr] = u < nu ? x : -INFINITY;
        }
      }
      float mx = (float)ell[ct][0];
#pragma unroll
      for (int rr = 1; rr < 4; ++rr) mx = fmaxf(mx, (float)ell[ct][rr]);
      mx = fmaxf(mx, xor16(mx));
      mx = fmaxf(mx, xor32(mx));
      if (lg == 0) sm.mx[w][16 * ct + li] = (double)mx;
    }
    __syncthreads();
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      const int col = 16 * ct + li, r = 64 * cg + col;
      double tmx = sm.mx[0][col];
#pragma unroll
      for (int x = 1; x < 4; ++x) tmx = fmax(tmx, sm.mx[x][col]);
      float e[4];
      double sum = 0.0;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        e[rr] = exp_mass(ell[ct][rr], tmx);
        sum += (double)e[rr];
      }
      if (r < R)
        *reinterpret_cast<float4*>(e_vals + ((int64_t)bh * R + r) * nbp + u_lane) =
            make_float4(e[0], e[1], e[2], e[3]);
      sum += xor16(sum);
      sum += xor32(sum);
      if (lg == 0) sm.sum[w][col] = sum;
    }
    __syncthreads();
    if (tid < 64 && 64 * cg + tid < R) {
      double mx = sm.mx[0][tid], sum = sm.sum[0][tid];
#pragma unroll
      for (int x = 1; x < 4; ++x) {
        mx = fmax(mx, sm.mx[x][tid]);
        sum += sm.sum[x][tid];
      }
      double2* tp = reinterpret_cast<double2*>(tile_part) +
                    ((int64_t)bh * R + 64 * cg + tid) * m.n_tiles + tile;
      *tp = make_double2(mx, sum);
    }
  }
}

// ----------------------------------------------------------- selection
// The decode's selection, per query; a query whose blocks all fit in k needs
// no scores. A query whose cutoff separates two scores closer than its tie_span
// is not selected but put on a list: prefill_rescore_kernel takes its block
// masses again with the decode's arithmetic, and a second launch of this
// kernel selects the listed queries from those, so that what the rounding of
// the scoring kernel could decide is decided as the decode decides it.
// SWN: tile weights (tiles x heads) in LDS, sized to the shape so that several
// workgroups share a compute unit. Past 32 queries per compute unit each
// workgroup takes a run of them (one per query spends 14 us per 16000 queries
// on starting workgroups alone, which is most of it where every block is
// selected).
//
// The span. With u = 2^-24, mean mu and variance v of a unit and x = s^2 <q^2, v>
// / 2, the two scorings' log masses differ by the rounding of their partial sums
// of s q . mu, at most u s |q| |mu| or so, and of the logarithms of n and 1 + x.
// Measured over 11 million units (d = 64 and 128, blocks and windows, means of
// up to 4700 = s |q| |mu|, x of up to e^11): at most 0.91 u (s |q| |mu| + 4 ln(1 +
// x) + 4), and this scoring no further from 64 bits than the decode's. That much
// (0.91 taken as 1, with the largest |mu| and v of the sequence and KV head) can
// move a mass and its head's normaliser, of each of the two scores. (Atomic maxima
// in place of a maximum per tile, reduced here, took the scoring of 8192 windows
// from 156 to 257 us.)
__device__ __forceinline__ float tie_span(float s, float q_norm2, float mu_norm2, float var) {
  const float ln = __builtin_amdgcn_logf(1.0f + 0.5f * s * s * q_norm2 * var) * kLn2f32;
  return fminf(1.0f, 0x1p-22f * (s * sqrtf(q_norm2 * mu_norm2) + 4.0f * ln + 4.0f));
}

struct PrefSelectArgs {
  Dims m;
  int T;
  const int32_t* seq_lens;
  const float* e_vals;
  const double* tile_part;
  int32_t *sel_ws, *sel_out;
  int32_t* near;           // NearLists
  const float2* unit_max;  // largest |mean|^2 and variance of each 16 units
  const float* q_norm2;    // |q|^2 per query row
  float s;
  int listed;  // select the listed queries (else every query, listing some)
  int exact;   // the masses have the decode's sums already: list none
};

template <int R, bool WIN, int NT, int SWN, int GMAX>
__global__ __launch_bounds__(NT) void prefill_select_kernel(PrefSelectArgs a) {
  __shared__ SelectSmem<NT, SWN> sm;
  __shared__ float wsc[WIN ? kMaxWindows : 1];
  __shared__ float2 s_um;  // (in LDS, as the span is: registers are short in the selection)
  __shared__ float s_span;
  const Dims& m = a.m;
  auto length = [&](int vh) {
    int L0, nv;
    chunk_bounds(m, a.seq_lens, vh / a.T / m.hkv, a.T, &L0, &nv);
    return L0 + min(vh % a.T + 1, nv);
  };
  // this workgroup's queries: a run of them, those whose blocks all fit in k
  // first, as one run of stores; or every gridDim.x-th entry of the lists, entry
  // x / bh of the list of x % bh (short lists spread over the workgroups)
  const NearLists nl = near_lists(m, a.near);
  const int n_q = m.bh * a.T, per = (n_q - 1) / (int)gridDim.x + 1;
  const int x0 = a.listed ? (int)blockIdx.x : (int)blockIdx.x * per;
  const int x1 = a.listed ? m.bh * *nl.longest : min(x0 + per, n_q);
  const int step = a.listed ? (int)gridDim.x : 1;
  if (x0 >= x1) return;
  if (!a.listed && per > 1) {
    for (int x = threadIdx.x; x < (x1 - x0) * m.k; x += NT) {
      const int vh = x0 + x / m.k, e = x % m.k, nb = (length(vh) + m.B - 1) / m.B;
      if (nb <= m.k) {
        a.sel_ws[(int64_t)vh * m.k + e] = e < nb ? e : -1;
        if (a.sel_out)
          a.sel_out[((int64_t)(vh % a.T) * m.bh + vh / a.T) * m.k + e] = e < nb ? e : -1;
      }
    }
    // (lengths grow along a run of one (sequence, KV head))
    if (x0 / a.T == (x1 - 1) / a.T && (length(x1 - 1) + m.B - 1) / m.B <= m.k) return;
  }
  int bh_max = -1;  // (sequence, KV head) whose largest |mean|^2 and variance s_um holds
  for (int x = x0; x < x1; x += step) {
    int vh = x;
    if (a.listed) {
      if (x / m.bh >= nl.count[x % m.bh]) continue;  // uniform
      vh = x % m.bh * a.T + nl.list[(int64_t)(x % m.bh) * a.T + x / m.bh];
    }
    const int bh = vh / a.T, i = vh % a.T, L = length(vh);
    if (!a.listed && per > 1 && (L + m.B - 1) / m.B <= m.k) continue;  // uniform; written above
    float span = 0.f;
    if (!a.listed && !a.exact && (L + m.B - 1) / m.B > m.k) {  // uniform
      if (bh != bh_max) {
        int L0, nv;
        chunk_bounds(m, a.seq_lens, bh / m.hkv, a.T, &L0, &nv);
        const int n16 = ((L0 + nv - 1) / m.us / kTileBlocks + 1) * 4;  // of the tiles scored
        float2 um = make_float2(0.f, 0.f);
        for (int t = threadIdx.x & 63; t < n16; t += 64) {
          const float2 v = a.unit_max[(int64_t)bh * m.n_tiles * 4 + t];
          um = make_float2(fmaxf(um.x, v.x), fmaxf(um.y, v.y));
        }
        s_um = make_float2(wave_max(um.x), wave_max(um.y));  // the same in every wavefront
        bh_max = bh;
      }
      float n2 = 0.f;
      for (int g = 0; g < m.group; ++g) n2 = fmaxf(n2, a.q_norm2[(int64_t)vh * m.group + g]);
      span = tie_span(a.s, n2, s_um.x, s_um.y);
    }
    s_span = span;  // the same in every thread, here and before barriers in the selection
    const bool near = select_blocks<NT, R, SWN, false, 0, WIN, GMAX, false, true>(
        m, vh, L, a.e_vals, a.tile_part, sm, a.sel_ws + (int64_t)vh * m.k, nullptr,
        a.sel_out ? a.sel_out + ((int64_t)i * m.bh + bh) * m.k : nullptr, wsc, &s_span);
    if (near && threadIdx.x == 0) {
      const int j = atomicAdd(nl.count + bh, 1);
      nl.list[(int64_t)bh * a.T + j] = i;
      atomicMax(nl.longest, j + 1);
    }
    __syncthreads();  // the next query's selection writes the same LDS
  }
}

// The block masses of the listed queries (Eqs. 8 and 10) with the decode's
// sums: v_mfma_f32_16x16x4_f32 adds its four products to the accumulator one
// fused multiply-add at a time in coordinate order, so two of them are the
// decode's eight-coordinate fp32 partial sum bit for bit, and those partials
// are added in fp64. One workgroup per (statistics tile, share of the list,
// sequence x KV head), wavefront w taking units 16 w .. 16 w + 15 as rows
// (operands straight from the statistics: lane holds unit lane % 16, coordinate
// 4 j + lane / 16 of k-step j), kept in registers; the columns are the heads of
// as many listed queries as 16 hold (kP), their coefficients staged in LDS.
// Where blocks repeat, every query can be listed (ties at the cutoff): 8192
// queries over 32 tiles of 64 blocks took 7400 us with one query's G columns at
// a time, 820 with kP.
// kAll: every query, in place of prefill_score_kernel (exact_scores); kAllOneTile:
// they fill one column tile at most, so the statistics are read quarter by quarter
// instead of kept (156 registers instead of 256, three workgroups per compute unit
// instead of two: 4 x 8 units of 2048 blocks 28 -> 23 us).
enum { kListed, kAll, kAllOneTile };

// Whether a chunk's queries are scored with the decode's sums at once, which takes
// 16 columns at a time but no listing, rescoring and second selection (two
// launches, and where many are listed more than the first): up to two tiles of
// columns, up to one workgroup's worth of work per place on the chip, and with
// strided windows, where blocks that share their best window tie and most queries
// are listed, up to eight. Score and selections, us, listing against at once:
// 4 x 8 units of 2048 blocks, 1 / 2 / 4 / 8 column tiles 57 / 65 / 68 / 87 against
// 33 / 52 / 77 / 123; 8 units of 128 blocks, 4 / 8 / 16 tiles 26 / 24 / 26 against
// 20 / 25 / 37; 4 x 8 units of 2048 windows, 1 / 4 / 8 / 16 tiles 80 / 125 / 195 /
// 328 against 42 / 109 / 187 / 343.
static bool exact_scores(const Dims& m, int T) {
  const int64_t n_ct = ceil_div(T, 16 / m.group);
  return n_ct <= (windowed(m) ? 8 : 2) ||
         n_ct * m.n_tiles * m.bh <= 2 * (int64_t)compute_units();
}

template <int D, int WHICH>
__global__ __launch_bounds__(256, WHICH == kAllOneTile ? 3 : 2) void prefill_rescore_kernel(
    Dims m, int T_, int W, const float* __restrict__ stats, const int32_t* __restrict__ seq_lens,
    const bf16_t* __restrict__ q, double s, int first_order, const double* __restrict__ ell_part,
    int32_t* __restrict__ near, float* __restrict__ e_vals, double* __restrict__ tile_part) {
  constexpr int NK = D / 4, NQ = D / 32;  // k-steps, partials per quarter of the coordinates
  constexpr bool ALL = WHICH != kListed, ONE = WHICH == kAllOneTile;
  __shared__ float s_c[2][NK][64];        // s q and s^2 q^2 / 2, as operands
  __shared__ double s_mx[4][16], s_sum[4][16];
  const int G = m.group, kP = 16 / G, nbp = m.n_tiles * kTileBlocks;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const NearLists nl = near_lists(m, near);
  const int tile = blockIdx.x, bh = blockIdx.z, n_near = ALL ? T_ : nl.count[bh];
  if ((int)blockIdx.y * kP >= n_near) return;
  int L0, nv;
  chunk_bounds(m, seq_lens, bh / m.hkv, T_, &L0, &nv);
  if (tile * kTileBlocks * m.us >= L0 + nv) return;  // past every query's tokens
  if (ALL && (L0 + nv + m.B - 1) / m.B <= m.k) return;  // every query selects every block
  auto position = [&](int x) { return ALL ? x : nl.list[(int64_t)bh * T_ + x]; };
  float pm[NK], pv[NK];
  const float* st = stats + stats_off4(m, bh, (int64_t)tile * kTileBlocks, 0, 0);  // uniform
  const float* st2 = first_order ? st : st + D / 4 * kTileBlocks * 4;
  auto load = [&](int qt) {  // a quarter of the coordinates
    const uint32_t o = (uint32_t)(16 * w + li) * 4u + (uint32_t)lg;
#pragma unroll
    for (int j = 2 * NQ * qt; j < 2 * NQ * (qt + 1); ++j) {
      pm[j] = (st + j * kTileBlocks * 4)[o];
      pv[j] = (st2 + j * kTileBlocks * 4)[o];
    }
  };
  auto quarter = [](int qp) { return qp / 2 + 2 * (qp % 2); };
#pragma unroll
  for (int qp = 0; qp < (ONE ? 1 : 4); ++qp) load(quarter(qp));
  const int u_lane = tile * kTileBlocks + 16 * w + 4 * lg;  // this lane's first result row
  for (int x0 = (int)blockIdx.y * kP; x0 < n_near; x0 += (int)gridDim.y * kP) {
    const int nc = min(kP, n_near - x0) * G;  // columns in use
    {
      const int c = min(li, nc - 1), g = c % G;
      const bf16_t* qr = q + (((int64_t)position(x0 + c / G) * m.batch + bh / m.hkv) * m.hq +
                              bh % m.hkv * G + g) * D + lg;
#pragma unroll
      for (int jj = 0; jj < NK / 4; ++jj) {
        const int j = 4 * jj + w;
        const double xq = (double)bf16_to_f32(qr[4 * j].bits);
        s_c[0][j][lane] = (float)(s * xq);
        s_c[1][j][lane] = (float)(0.5 * s * s * xq * xq);
      }
    }
    __syncthreads();
    double am[2][4], av[2][4];  // quarters qt and qt + 2 of the coordinates added, result row
#pragma unroll
    for (int qp = 0; qp < 4; ++qp) {
      const int qt = quarter(qp);
      if (ONE && qp < 3) load(quarter(qp + 1));
      double dm[4] = {0.0, 0.0, 0.0, 0.0}, dv[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int jp = 0; jp < NQ; ++jp) {
        floatx4 pa = {0.f, 0.f, 0.f, 0.f}, pb = pa;
#pragma unroll
        for (int y = 0; y < 2; ++y) {
          const int j = 2 * (NQ * qt + jp) + y;
          pa = __builtin_amdgcn_mfma_f32_16x16x4f32(pm[j], s_c[0][j][lane], pa, 0, 0, 0);
          pb = __builtin_amdgcn_mfma_f32_16x16x4f32(pv[j], s_c[1][j][lane], pb, 0, 0, 0);
        }
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          dm[rr] += (double)pa[rr];
          dv[rr] += (double)pb[rr];
        }
      }
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        am[qp / 2][rr] = qp % 2 ? am[qp / 2][rr] + dm[rr] : dm[rr];
        av[qp / 2][rr] = qp % 2 ? av[qp / 2][rr] + dv[rr] : dv[rr];
      }
      __builtin_amdgcn_sched_barrier(0);  // (operands of one quarter at a time in registers)
    }
    // this lane's column: position i, head g of the group
    const int c = min(li, nc - 1), i = position(x0 + c / G), g = c % G;
    const int64_t vh = (int64_t)bh * T_ + i;
    const int L = L0 + min(i + 1, nv), nu = (L + m.us - 1) / m.us;
    double ell[4];
    float mx = -INFINITY;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int u = u_lane + rr, n = min(m.ul, max(L - u * m.us, 1));
      // the quarters in the order the decode adds them: (0 + 2) + (1 + 3)
      const double dm = am[0][rr] + am[1][rr], dv = av[0][rr] + av[1][rr];
      double e = log_mass(dm, n, (float)dv * __builtin_amdgcn_rcpf((float)n), first_order);
      const int wu = (L0 + i) / m.us - u;
      if (i < nv && wu >= 0 && wu < W) e = ell_part[(vh * W + wu) * G + g];
      ell[rr] = u < nu ? e : -INFINITY;
      mx = fmaxf(mx, (float)ell[rr]);
    }
    mx = fmaxf(mx, xor16(mx));
    mx = fmaxf(mx, xor32(mx));
    if (lg == 0) s_mx[w][li] = (double)mx;
    __syncthreads();
    double tmx = s_mx[0][li];
#pragma unroll
    for (int y = 1; y < 4; ++y) tmx = fmax(tmx, s_mx[y][li]);
    float e[4];
    double sum = 0.0;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      e[rr] = exp_mass(ell[rr], tmx);
      sum += (double)e[rr];
    }
    // (a tile past this position's tokens gets zeros, which nothing reads)
    if (li < nc)
      *reinterpret_cast<float4*>(e_vals + (vh * G + g) * nbp + u_lane) =
          make_float4(e[0], e[1], e[2], e[3]);
    sum += xor16(sum);
    sum += xor32(sum);
    if (lg == 0) s_sum[w][li] = sum;
    __syncthreads();
    if (tid < nc) {
      for (int y = 1; y < 4; ++y) sum = (y == 1 ? s_sum[0][tid] : sum) + s_sum[y][tid];
      double2* tp = reinterpret_cast<double2*>(tile_part) + (vh * G + g) * m.n_tiles + tile;
      *tp = make_double2(tmx, sum);
    }
    if (ONE) break;
  }
}

// ------------------------------------------------------ fused group pass
// One wavefront per (kP consecutive positions, sequence x KV head, split); the
// four of a workgroup take consecutive positions, or splits of the same ones
// (prefill_positions, prefill_splits, prefill_wg_groups). The kP G query rows
// are the columns of the wavefront's matrix-core tiles
// (16 at most), and it walks once over the union of the blocks its positions
// select, one 32-token step at a time, with keys and values straight in
// registers (the bf16 caches hold a step in operand order):
//   exact    S = K q, masked per column to the blocks its position selected
//            and to the tokens it sees, online softmax, O += V^T P
//   linear   W = phi(K) phi(q), masked the same way, R += V^T W
// so keys, values and phi(k) (the exponentials, the largest share of the
// arithmetic) are shared by kP queries, and no product column is idle at
// G = 4. The residual of Eq. 14 starts from -phi(q) S_x, S_x being S_bar
// before the block x of the wavefront's positions (which lie in one block:
// they are aligned to their number in the sequence). Tokens of that block
// from position tb = max(start of the block, L0) on are not in S_x, so there
// a selected block's linear terms cancel and are left out, and an unselected
// one's enter with weight -1. Nothing of the linear branch is formed where
// every block is selected (the residual is zero) or without it.
// Not split: the output rows are finished from the registers. Split: split
// s takes every n_split-th block of the union and writes one record per
// query, merged by prefill_merge_kernel.
// A weight of zero does not hide an infinite or NaN value of a token that
// another position of the tile attends to: a wavefront whose sums end up not
// finite repeats its pass with each position multiplying only the tokens that
// count for it.
// ONE: one position per wavefront, which walks its selection as it is listed,
// without forming a union (4 x 8 units at 128K, 1 position 27 -> 20 us; 8 units at
// 200K in four segments 34 -> 21).
// One workgroup per query read each query's blocks anew: 138.5 us + 25.9 us
// for the linear branch for 32 positions at 128K tokens (8 KV heads, 4 heads
// each, D = 128, 64 blocks of 64), now 115.4 us with the linear branch in it
// (random queries: hardly a block is shared). A whole prefill of a prompt,
// where neighbours share most of their blocks, went from 4440 to 180 us, and
// one that continues 126K tokens from 2490 to 1145 us.
constexpr int kSegBlocks = 1024;  // block ids of one pass over the union

template <int D>
struct GroupSmem {  // of one wavefront
  uint4 q[3][D / 32][64];         // operands of its columns: q, phi(q) hi, phi(q) lo
  union {
    struct {
      uint32_t mask[kSegBlocks / 2];  // positions that selected each block (16 bits each)
      uint16_t list[kSegBlocks];      // blocks of the union, ascending
    };
    int32_t one[SPLA_MAX_TOP_K + 1];  // one position: the blocks it walks
  };
};

struct GroupArgs {
  Dims m;
  int T, P, n_blk, gw, n_grp, n_split, n_items, stride;
  float s, eps;
  uint32_t flags;
  const bf16_t *kc, *vc, *q;
  const int32_t *seq_lens, *sel, *table;
  const uint4 *s_hi, *s_lo;
  const float *z_pre, *gamma;
  float* part;
  bf16_t* out;
};

// Orders this wavefront's LDS accesses (the hardware keeps them in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// What a wavefront of the group pass keeps: its place and its sums.
template <int D>
struct GroupWave {
  floatx4 ax[D / 16], al[D / 16];  // exact and residual sums: coordinates 16 t + 4 lg .. + 3
  float m_run, l_run, zl;  // the column's max; this lane's share of its sum and of the
                           // residual normaliser
  int L0, nv, Lend;
  int i0, if0, il0;        // first position of the wavefront; first and last that exist
  int P, pc;               // positions per wavefront; this lane's position
  bool live;               // whether this lane's column exists
  int Lc;                  // tokens it sees
  int bw, tb;              // block of the positions, first token not in S_x
  int nbg, split;
};

// One walk over the union of the selections. LIN: with the linear branch.
// SLOW: each position multiplies only the tokens that count for it.
template <int D, int BLK, bool ONE, bool LIN, bool SLOW>
__device__ __forceinline__ void group_walk(const GroupArgs& a, int bh, GroupWave<D>& s,
                                           GroupSmem<D>& sm) {
  uint32_t* mask = sm.mask;
  uint16_t* list = sm.list;
  constexpr int KS = D / 32, MT = D / 16, CPB = BLK / 32;
  const Dims& m = a.m;
  const int lane = threadIdx.x & 63, lg = lane >> 4;
  const int32_t* sp = a.sel + ((int64_t)bh * a.T + s.if0) * m.k;
  for (int seg = 0; seg < (ONE ? 1 : s.nbg); seg += kSegBlocks) {
    int n_list = 0;
    if constexpr (ONE) {
      // ---- one position: its selection, 2 block + 1, and 2 block for its own
      // block where that is walked without being selected
      bool own = false;
      for (int x0 = 0; x0 < m.k; x0 += 64) {
        const int id = x0 + lane < m.k ? sp[x0 + lane] : -1;
        if (id >= 0) sm.one[x0 + lane] = 2 * id + 1;
        n_list += __popcll(__ballot(id >= 0));  // (the entries that are there come first)
        own |= __ballot(id == s.bw) != 0ull;
      }
      if (LIN && !own) {
        if (lane == 0) sm.one[n_list] = 2 * s.bw;
        ++n_list;
      }
      wave_lds_fence();
    } else {
      // ---- the union of the positions' selections within this segment
      const int ns = min(kSegBlocks, s.nbg - seg);
      for (int x = lane; 2 * x < ns; x += 64) mask[x] = 0u;
      wave_lds_fence();
      {
        for (int x = lane; x < (s.il0 - s.if0 + 1) * m.k; x += 64) {
          const int id = sp[x] - seg, pos = s.if0 - s.i0 + x / m.k;
          if (id >= 0 && id < ns) atomicOr(&mask[id >> 1], 1u << (pos + 16 * (id & 1)));
        }
      }
      wave_lds_fence();
      for (int x0 = 0; x0 < ns; x0 += 128) {  // two blocks per lane
        const int x = x0 + 2 * lane;
        const uint32_t v = x < ns ? mask[x >> 1] : 0u;
        // with the linear branch the positions' own block is always walked
        const bool p0 = (v & 0xFFFFu) || (LIN && seg + x == s.bw);
        const bool p1 = (v >> 16) || (LIN && seg + x + 1 == s.bw);
        const uint32_t n = (p0 ? 1u : 0u) + (p1 ? 1u : 0u);
        const uint32_t incl = wave_incl_scan_u32(n);
        int pos = n_list + (int)(incl - n);
        if (p0) list[pos++] = (uint16_t)x;
        if (p1) list[pos] = (uint16_t)(x + 1);
        n_list += (int)lane_u32(incl, 63);
      }
      wave_lds_fence();
    }
    const int n_mine = n_list > s.split ? (n_list - s.split + a.n_split - 1) / a.n_split : 0;
    const int n_steps = n_mine * CPB;
    if (n_steps == 0) continue;
    auto entry = [&](int st) {
      const int at = s.split + (st / CPB) * a.n_split;
      return __builtin_amdgcn_readfirstlane(ONE ? sm.one[at] : (int)list[at]);
    };
    auto block = [&](int x) { return ONE ? x >> 1 : seg + x; };
    auto slot0 = [&](int st, int x) {  // first element of step st, of entry x
      int64_t slot = (int64_t)bh * m.nb_cap + block(x);
      if (a.table) {
        const int pg = block_page(m, a.table, bh, block(x));
        slot = (int64_t)(pg < 0 ? 0 : pg) * m.hkv + bh % m.hkv;
      }
      return (slot * BLK + (st % CPB) * 32) * D;
    };
    bf16x8 ka[2][KS], va[MT];
    auto load_k = [&](int64_t e0) {
      const bf16x8* kp = reinterpret_cast<const bf16x8*>(a.kc + e0) + lane;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ka[mt][ks] = kp[(mt * KS + ks) * 64];
    };
    auto load_v = [&](int64_t e0) {
      const bf16x8* vp = reinterpret_cast<const bf16x8*>(a.vc + e0) + lane;
#pragma unroll
      for (int t = 0; t < MT; ++t) va[t] = vp[t * 64];
    };
    int x = entry(0);
    int64_t e0 = slot0(0, x);
    load_k(e0);
    load_v(e0);
    for (int st = 0; st < n_steps; ++st) {
      const int id = block(x), base = id * BLK + (st % CPB) * 32;
      const uint32_t bits =
          ONE ? (uint32_t)(x & 1)
              : (uint32_t)__builtin_amdgcn_readfirstlane((int)(mask[x >> 1] >> (16 * (x & 1)))) &
                    ((1u << s.P) - 1u);
      // the next step: its keys are loaded when this step's are used up
      const int nx = st + 1 < n_steps ? st + 1 : st;
      x = entry(nx);
      e0 = slot0(nx, x);
      const bool sel = s.live && ((bits >> s.pc) & 1u);
      const bool cur = id == s.bw;
      const int nvis = s.Lc - base;  // tokens of the step this column sees
      bf16x8 eh, el, wh, wl;
      // the operands of the columns come from LDS k-step by k-step; the offset
      // is opaque so that the loads stay in the loop (in registers throughout
      // they would push others out to scratch memory)
      int qo = lane;
      asm volatile("" : "+v"(qo));
      auto operand = [&](int x, int ks) {
        return __builtin_bit_cast(bf16x8, sm.q[x][ks][qo]);
      };
      // exact logits
      floatx4 sx[2];
      sx[0] = sx[1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 qx = operand(0, ks);
        sx[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[0][ks], qx, sx[0], 0, 0, 0);
        sx[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[1][ks], qx, sx[1], 0, 0, 0);
      }
      if constexpr (LIN) {
        // linear weights: exp(k - max k) k-step by k-step, straight into its
        // products; each lane sums its part of its key row (row lane % 16 of
        // the tile), and 1 / sum is applied to the result rows
        floatx4 sl[2];
        float zinv[2];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          sl[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
          float mx = -INFINITY;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) mx = fmaxf(mx, (float)ka[mt][ks][e]);
          mx = fmaxf(mx, xor16(mx));
          mx = fmaxf(mx, xor32(mx));
          const float mxl = mx * kLog2e;
          float sum = 0.f;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            float f[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              f[e] = __builtin_amdgcn_exp2f(fmaf((float)ka[mt][ks][e], kLog2e, -mxl));
              sum += f[e];
            }
            bf16x8 fh, fl;
            split_bf16x8(f, fh, fl);
            const bf16x8 qh = operand(1, ks), ql = operand(2, ks);
            sl[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fl, qh, sl[mt], 0, 0, 0);
            sl[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh, ql, sl[mt], 0, 0, 0);
            sl[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fh, qh, sl[mt], 0, 0, 0);
          }
          sum += xor16(sum);
          sum += xor32(sum);
          zinv[mt] = 1.0f / sum;
        }
        float wv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int tt = 8 * lg + e;         // token of the step
          const bool in = base + tt < s.tb;  // in S_x
          const float zi = __shfl(zinv[e >> 2], 4 * lg + (e & 3), kWave);
          const float wt = sl[e >> 2][e & 3] * zi;
          float v = in ? (sel ? wt : 0.f) : (cur && !sel ? -wt : 0.f);
          v = tt < nvis ? v : 0.f;
          wv[e] = v;
          s.zl += v;
        }
        split_bf16x8(wv, wh, wl);
      }
      load_k(e0);
      // online softmax of the exact columns
      float xv[8], cmax = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xv[e] = sel && 8 * lg + e < nvis ? sx[e >> 2][e & 3] * a.s : -INFINITY;
        cmax = fmaxf(cmax, xv[e]);
      }
      cmax = fmaxf(cmax, xor16(cmax));
      cmax = fmaxf(cmax, xor32(cmax));
      const float mn = fmaxf(s.m_run, cmax);
      if (__ballot(mn > s.m_run) != 0ull) {
        const float alpha = s.m_run == -INFINITY ? 0.f : __expf(s.m_run - mn);
        s.l_run *= alpha;
#pragma unroll
        for (int t = 0; t < MT; ++t) s.ax[t] = s.ax[t] * alpha;
        s.m_run = mn;
      }
      const float ms = s.m_run == -INFINITY ? 0.f : s.m_run;
      float pv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pv[e] = __builtin_amdgcn_exp2f((xv[e] - ms) * kLog2e);
        s.l_run += pv[e];
      }
      split_bf16x8(pv, eh, el);
      if (base + 32 > s.Lend) {  // rows past the tokens may hold anything: zero them
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (base + 8 * lg + e >= s.Lend) va[t][e] = (__bf16)0.f;
      }
      if constexpr (!SLOW) {
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          s.ax[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t], eh, s.ax[t], 0, 0, 0);
          s.ax[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t], el, s.ax[t], 0, 0, 0);
          if constexpr (LIN) {
            s.al[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t], wh, s.al[t], 0, 0, 0);
            s.al[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t], wl, s.al[t], 0, 0, 0);
          }
        }
      } else {
#pragma unroll 1
        for (int p = s.if0 - s.i0; p <= s.il0 - s.i0; ++p) {
          const int np = s.L0 + min(s.i0 + p + 1, s.nv) - base;  // tokens position p sees
          const bool ps = (bits >> p) & 1u, mine = s.pc == p;
          uint32_t mx = 0u, mw = 0u;  // this lane's tokens that count for p
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const bool in = base + 8 * lg + e < s.tb, see = 8 * lg + e < np;
            mx |= (uint32_t)(see & ps) << e;
            mw |= (uint32_t)(see & (in ? ps : cur & !ps)) << e;
          }
#pragma unroll
          for (int t = 0; t < MT; ++t) {
            bf16x8 vx = va[t], vw = va[t];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              if (!((mx >> e) & 1u)) vx[e] = (__bf16)0.f;
              if (!((mw >> e) & 1u)) vw[e] = (__bf16)0.f;
            }
            floatx4 x4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vx, eh, s.ax[t], 0, 0, 0);
            x4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vx, el, x4, 0, 0, 0);
            s.ax[t] = mine ? x4 : s.ax[t];
            if constexpr (LIN) {
              x4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vw, wh, s.al[t], 0, 0, 0);
              x4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vw, wl, x4, 0, 0, 0);
              s.al[t] = mine ? x4 : s.al[t];
            }
          }
        }
      }
      load_v(e0);
    }
  }
}

// The sums before any block: zero, or minus the global term (LIN): al = -S_x^T
// phi(q), zl = -<phi(q), z_x>, x the xw-th block of the chunk. Its coordinate
// tiles are dealt out over the splits (in one of them they took as long as four
// to six steps), zl is split 0's.
template <int D, bool LIN>
__device__ __forceinline__ void group_start(const GroupArgs& a, int bh, int xw, GroupWave<D>& s,
                                            const GroupSmem<D>& sm) {
  constexpr int KS = D / 32, MT = D / 16;
  const int lane = threadIdx.x & 63, lg = lane >> 4;
  s.m_run = -INFINITY;
  s.l_run = s.zl = 0.f;
#pragma unroll
  for (int t = 0; t < MT; ++t) s.ax[t] = s.al[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  if constexpr (!LIN) return;
  const float* zp = a.z_pre + ((int64_t)bh * a.n_blk + xw) * D + 8 * lg;
  const uint4* sh = a.s_hi + ((int64_t)bh * a.n_blk + xw) * (D * D / 8) + lane;
  const uint4* sl = a.s_lo + ((int64_t)bh * a.n_blk + xw) * (D * D / 8) + lane;
  if (s.split == 0) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 qh = __builtin_bit_cast(bf16x8, sm.q[1][ks][lane]);
      const bf16x8 ql = __builtin_bit_cast(bf16x8, sm.q[2][ks][lane]);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        s.zl = fmaf(-((float)qh[e] + (float)ql[e]), zp[32 * ks + e], s.zl);
    }
  }
  const int t0 = s.split < MT ? s.split : -1, ts = min(a.n_split, MT);
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    if (t % ts != t0) continue;  // uniform
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 qh = __builtin_bit_cast(bf16x8, sm.q[1][ks][lane]);
      const bf16x8 ql = __builtin_bit_cast(bf16x8, sm.q[2][ks][lane]);
      const bf16x8 ah = __builtin_bit_cast(bf16x8, sh[(t * KS + ks) * 64]);
      const bf16x8 aw = __builtin_bit_cast(bf16x8, sl[(t * KS + ks) * 64]);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, qh, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, ql, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, qh, acc, 0, 0, 0);
    }
    s.al[t] = -acc;
  }
}

// Whether any live column's sums are infinite or NaN.
template <int D>
__device__ __forceinline__ bool group_not_finite(const GroupWave<D>& s) {
  bool bad = false;
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      bad = bad | !(fabsf(s.ax[t][r]) < INFINITY) | !(fabsf(s.al[t][r]) < INFINITY);
  return __ballot(bad && s.live) != 0ull;
}

template <int D, int BLK, bool ONE>
__global__ __launch_bounds__(256, 2) void prefill_group_kernel(GroupArgs a) {
  constexpr int KS = D / 32, MT = D / 16;
  __shared__ GroupSmem<D> lds[4];
  const Dims& m = a.m;
  const int per = (int)(gridDim.x / 8);
  const int item = ((int)blockIdx.x % 8) * per + (int)blockIdx.x / 8;  // one XCD: one run of items
  if (item >= a.n_items) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int gw = a.gw, wg_splits = a.n_split * gw / 4;  // workgroups that share gw groups
  const int split = item % wg_splits * (4 / gw) + w / gw, gq = item / wg_splits;
  const int bh = gq / a.n_grp, gi = a.n_grp - 1 - gq % a.n_grp;  // longest prefixes first
  const int b = bh / m.hkv, h = bh % m.hkv, G = m.group, T = a.T;
  const int c = lane & 15, lg = lane >> 4;
  GroupSmem<D>& sm = lds[w];
  GroupWave<D> s;
  const int P = ONE ? 1 : a.P;
  s.P = P;
  s.split = split;
  chunk_bounds(m, a.seq_lens, b, T, &s.L0, &s.nv);
  const int L0 = s.L0, nv = s.nv;
  // chunk positions of the wavefront (aligned in the sequence): i0 .. i0 + P - 1
  const int i0 = (L0 / (gw * P) + gi) * gw * P + P * (w % gw) - L0;
  if (i0 >= T || i0 + P <= 0) return;
  const int if0 = max(i0, 0), il0 = min(i0 + P, T) - 1;
  s.i0 = i0;
  s.if0 = if0;
  s.il0 = il0;
  s.Lend = L0 + nv;
  const int Ll = L0 + min(il0 + 1, nv);
  s.nbg = (Ll + BLK - 1) / BLK;
  const bool rla = !(a.flags & SPLA_FLAG_NO_RLA);
  const bool lin = rla && s.nbg > m.k;  // the last position sees the most blocks

  // this lane's column: query row (position i, head g)
  const int pc = c / G, g = c - pc * G, i = i0 + pc;
  const bool live = pc < P && i >= 0 && i < T;
  s.pc = pc;
  s.live = live;
  s.Lc = live ? L0 + min(i + 1, nv) : 0;
  const bool all_sel = (s.Lc + BLK - 1) / BLK <= m.k;
  s.bw = (i0 < nv ? L0 + if0 : m.cap - 1) / BLK;
  s.tb = max(s.bw * BLK, L0);
  const int xw = max(0, s.bw - L0 / BLK);  // S_x among the chunk's blocks
  {
    const bf16_t* qr =
        a.q + (((int64_t)(live ? i : if0) * m.batch + b) * m.hq + h * G + (live ? g : 0)) * D + 8 * lg;
    const uint32_t msk = live ? 0xFFFFFFFFu : 0u;
    bf16x8 qx[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 r = *reinterpret_cast<const uint4*>(qr + 32 * ks);
      const uint4 x = make_uint4(r.x & msk, r.y & msk, r.z & msk, r.w & msk);
      sm.q[0][ks][lane] = x;
      qx[ks] = __builtin_bit_cast(bf16x8, x);
    }
    float mx = -INFINITY, sum = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) mx = fmaxf(mx, (float)qx[ks][e]);
    mx = fmaxf(mx, xor16(mx));
    mx = fmaxf(mx, xor32(mx));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) sum += __expf((float)qx[ks][e] - mx);
    sum += xor16(sum);
    sum += xor32(sum);
    const float inv = live ? 1.0f / sum : 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      float f[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] = __expf((float)qx[ks][e] - mx) * inv;
      bf16x8 hi, lo;
      split_bf16x8(f, hi, lo);
      sm.q[1][ks][lane] = __builtin_bit_cast(uint4, hi);
      sm.q[2][ks][lane] = __builtin_bit_cast(uint4, lo);
    }
  }
  wave_lds_fence();
  if (lin) {
    group_start<D, true>(a, bh, xw, s, sm);
    group_walk<D, BLK, ONE, true, false>(a, bh, s, sm);
  } else {
    group_start<D, false>(a, bh, xw, s, sm);
    group_walk<D, BLK, ONE, false, false>(a, bh, s, sm);
  }
  if (group_not_finite<D>(s)) {
    if (lin) {
      group_start<D, true>(a, bh, xw, s, sm);
      group_walk<D, BLK, ONE, true, true>(a, bh, s, sm);
    } else {
      group_start<D, false>(a, bh, xw, s, sm);
      group_walk<D, BLK, ONE, false, true>(a, bh, s, sm);
    }
  }
  auto& ax = s.ax;
  auto& al = s.al;
  float m_run = s.m_run, l_run = s.l_run, zl = s.zl;

  // ---- the columns' results
  l_run += xor16(l_run);
  l_run += xor32(l_run);
  zl += xor16(zl);
  zl += xor32(zl);
  if (!live) return;
  if (a.n_split > 1) {
    float* rec = a.part + (((int64_t)bh * T + i) * a.n_split + split) * a.stride;
    if (lg == 0) {
      rec[g] = m_run;
      rec[16 + g] = l_run;
      rec[32 + g] = -zl;
    }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      *reinterpret_cast<floatx4*>(rec + kPartHead + g * D + 16 * t + 4 * lg) = ax[t];
      *reinterpret_cast<floatx4*>(rec + kPartHead + (G + g) * D + 16 * t + 4 * lg) = -al[t];
    }
    return;
  }
  const bool res = rla && !all_sel;
  const float rden = (a.flags & SPLA_FLAG_RLA_NORMALIZE) ? 1.f / zl : -1.f;  // both negated
  float ss = 0.f;
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      al[t][r] = res ? al[t][r] * rden : 0.f;
      ss += al[t][r] * al[t][r];
    }
  ss += xor16(ss);
  ss += xor32(ss);
  const float inv = 1.0f / sqrtf(ss / D + a.eps), rl = 1.0f / l_run;
  const float* gm = a.gamma + (int64_t)(h * G + g) * D + 4 * lg;
  const int64_t orow = (((int64_t)i * m.batch + b) * m.hq + h * G + g) * D + 4 * lg;
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    float o[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float x = ax[t][r] * rl;
      o[r] = res ? fmaf(gm[16 * t + r] * al[t][r], inv, x) : x;
    }
    const bf16x2 o0 = __builtin_convertvector(f32x2{o[0], o[1]}, bf16x2);
    const bf16x2 o1 = __builtin_convertvector(f32x2{o[2], o[3]}, bf16x2);
    *reinterpret_cast<uint2*>(a.out + orow + 16 * t) =
        make_uint2(__builtin_bit_cast(uint32_t, o0), __builtin_bit_cast(uint32_t, o1));
  }
}

// ---------------------------------------------------------------- merge
// The records of a query whose blocks were split over n_rec workgroups.
template <int D>
__global__ __launch_bounds__(512) void prefill_merge_kernel(
    Dims m, int T_, float eps, uint32_t flags, const float* __restrict__ gamma,
    const int32_t* __restrict__ seq_lens, const float* __restrict__ part, int n_rec, int stride,
    bf16_t* __restrict__ out) {
  const int vh = blockIdx.x, bh = vh / T_, i = vh % T_;
  int L0, nv;
  chunk_bounds(m, seq_lens, bh / m.hkv, T_, &L0, &nv);
  const int L = L0 + min(i + 1, nv), nb = (L + m.B - 1) / m.B;
  merge_head<bf16_t, D, false>(m, eps, flags, gamma, nb <= m.k, L,
                               part + (int64_t)vh * n_rec * stride, n_rec, stride,
                               out + (int64_t)i * m.batch * m.hq * D, bh,
                               (int)(threadIdx.x >> 6));
}

// ------------------------------------------------------------- launcher
template <int R, bool WIN, int NT>
static void prefill_select_r(const PrefSelectArgs& a, hipStream_t st) {
  // tiles x heads: at most NT R / 64 tiles of blocks, kMaxWindows / 64 of windows
  constexpr int SWN = (WIN ? kMaxWindows / kTileBlocks : NT * R / kTileBlocks) * 8;
  auto kern = a.m.group <= 4 ? prefill_select_kernel<R, WIN, NT, SWN, 4>
                             : prefill_select_kernel<R, WIN, NT, SWN, 8>;
  const int64_t queries = (int64_t)a.m.bh * a.T;
  // (the listed queries are few as a rule: fewer workgroups to start)
  const int64_t most = (int64_t)compute_units() * (NT != 256 ? (a.listed ? 1 : 8) : (a.listed ? 4 : 32));
  hipLaunchKernelGGL(kern, dim3((unsigned)(queries < most ? queries : most)), dim3(NT), 0, st, a);
}

template <int D, int BLK>
static void prefill_group_db(const GroupArgs& a, hipStream_t st) {
  auto kern = a.P == 1 ? prefill_group_kernel<D, BLK, true> : prefill_group_kernel<D, BLK, false>;
  hipLaunchKernelGGL(kern, dim3((unsigned)align_up(a.n_items, 8)), dim3(256), 0, st, a);
}

template <int D>
static hipError_t prefill_chunk_d(const Dims& m, const spla_config& cfg, const spla_cache& c,
                                  int T, const bf16_t* k_new, const bf16_t* v_new,
                                  const bf16_t* q, const float* gamma, bf16_t* out,
                                  int32_t* sel_out, const PrefillWs& ws, char* base,
                                  const spla_events* ev, hipStream_t st) {
  const double s_score =
      cfg.softmax_scale > 0.f ? (double)cfg.softmax_scale : 1.0 / sqrt((double)m.d);
  const int fo = (cfg.flags & SPLA_FLAG_FIRST_ORDER) ? 1 : 0;
  const int lin = (cfg.flags & SPLA_FLAG_NO_RLA) ? 0 : 1;
  const int W = m.ul / m.us;
  const int n_blk = prefill_blocks(m, T);
  hipError_t e;
  // 1. log masses of the units in progress, from the statistics before the
  // chunk; then the chunk's K/V rows and the statistics of the units it touches
  mark_phase(ev, SPLA_PHASE_APPEND, false, st);
  hipLaunchKernelGGL((prefill_partial_kernel<D>),
                     dim3((unsigned)(ceil_div(T + m.ul, m.us) + 1), (unsigned)m.bh), dim3(256), 0,
                     st, m, T, W, (const float*)c.blk_stats, (const int32_t*)c.seq_lens, k_new, q,
                     s_score, fo, (double*)(base + ws.ell_part));
  if ((e = launch_append_blocks(m, c, k_new, v_new, T, nullptr, st, true)) != hipSuccess) return e;
  mark_phase(ev, SPLA_PHASE_APPEND, true, st);
  // 2. S_bar before each block the chunk touches; S_bar and z_bar past the chunk
  mark_phase(ev, SPLA_PHASE_LINEAR, false, st);
  if ((e = launch_block_states(m, c, k_new, v_new, T, n_blk, (float*)(base + ws.part_s),
                               (float*)(base + ws.part_z), st)) != hipSuccess)
    return e;
  hipLaunchKernelGGL((prefill_prefix_kernel<D>), dim3(D * D / 8 / 256, (unsigned)m.bh), dim3(256),
                     0, st, m, T, n_blk, lin, (const int32_t*)c.seq_lens,
                     (const float*)(base + ws.part_s), (const float*)(base + ws.part_z),
                     c.lin_state, c.lin_norm, (uint4*)(base + ws.s_hi), (uint4*)(base + ws.s_lo),
                     (float*)(base + ws.z_pre), (int32_t*)(base + ws.near));
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark_phase(ev, SPLA_PHASE_LINEAR, true, st);
  // 3. block scores of every query; the queries are split over more
  // workgroups where the tiles alone leave compute units idle. exact: with the
  // decode's sums at once, so that no query is listed
  mark_phase(ev, SPLA_PHASE_SCORE, false, st);
  const int64_t tiles = (int64_t)m.n_tiles * m.bh, n_cg = ceil_div((int64_t)T * m.group, 64);
  const int64_t n_ct = ceil_div(T, 16 / m.group);
  const bool exact = exact_scores(m, T);
  // (two workgroups per compute unit at a time, and as many again)
  const int64_t qs = ceil_div((exact ? 2 : 4) * (int64_t)compute_units(), tiles);
  auto rescore = [&](auto kern, int64_t most) {
    hipLaunchKernelGGL(kern, dim3((unsigned)m.n_tiles, (unsigned)(qs < most ? qs : most), (unsigned)m.bh),
                       dim3(256), 0, st, m, T, W, (const float*)c.blk_stats,
                       (const int32_t*)c.seq_lens, q, s_score, fo,
                       (const double*)(base + ws.ell_part), (int32_t*)(base + ws.near),
                       (float*)(base + ws.e_vals), (double*)(base + ws.tile_part));
  };
  if (exact)
    rescore(n_ct == 1 ? prefill_rescore_kernel<D, kAllOneTile> : prefill_rescore_kernel<D, kAll>,
            n_ct);
  else
    hipLaunchKernelGGL((prefill_score_kernel<D>),
                       dim3((unsigned)m.n_tiles, (unsigned)(qs < n_cg ? qs : n_cg), (unsigned)m.bh),
                       dim3(256), 0, st, m, T, W, (const float*)c.blk_stats,
                       (const int32_t*)c.seq_lens, q, s_score, fo,
                       (const double*)(base + ws.ell_part), (float*)(base + ws.e_vals),
                       (double*)(base + ws.tile_part), (float2*)(base + ws.unit_max),
                       (float*)(base + ws.q_norm2));
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark_phase(ev, SPLA_PHASE_SCORE, true, st);
  // 4. selection of every query: without windows and up to 2048 blocks, 256
  // threads with up to eight blocks each (four wavefronts: cheaper barriers
  // and histogram scans; 32 positions at 128K 21.2 -> 17.5 us); otherwise
  // blocks per thread of a 1024-thread workgroup
  mark_phase(ev, SPLA_PHASE_SELECT, false, st);
  const int per = (int)ceil_div(m.nb_cap, kPrefSelThreads);
  PrefSelectArgs sa;
  sa.m = m;
  sa.T = T;
  sa.seq_lens = c.seq_lens;
  sa.e_vals = (const float*)(base + ws.e_vals);
  sa.tile_part = (const double*)(base + ws.tile_part);
  sa.sel_ws = (int32_t*)(base + ws.sel);
  sa.sel_out = sel_out;
  sa.near = (int32_t*)(base + ws.near);
  sa.unit_max = (const float2*)(base + ws.unit_max);
  sa.q_norm2 = (const float*)(base + ws.q_norm2);
  sa.s = (float)s_score;
  sa.listed = 0;
  sa.exact = exact;
  auto select = [&](auto f) {
    f(sa, st);
    if (exact) return;
    sa.listed = 1;
    rescore(prefill_rescore_kernel<D, kListed>, n_cg);
    f(sa, st);
  };
  if (windowed(m)) {
    if (per <= 1) select(prefill_select_r<1, true, kPrefSelThreads>);
    else if (per <= 2) select(prefill_select_r<2, true, kPrefSelThreads>);
    else if (per <= 4) select(prefill_select_r<4, true, kPrefSelThreads>);
    else if (per <= 8) select(prefill_select_r<8, true, kPrefSelThreads>);
    else select(prefill_select_r<16, true, kPrefSelThreads>);
  } else {
    if (m.nb_cap <= 256) select(prefill_select_r<1, false, 256>);
    else if (m.nb_cap <= 512) select(prefill_select_r<2, false, 256>);
    else if (m.nb_cap <= 1024) select(prefill_select_r<4, false, 256>);
    else if (m.nb_cap <= 2048) select(prefill_select_r<8, false, 256>);
    else if (per <= 4) select(prefill_select_r<4, false, kPrefSelThreads>);
    else if (per <= 8) select(prefill_select_r<8, false, kPrefSelThreads>);
    else if (per <= 16) select(prefill_select_r<16, false, kPrefSelThreads>);
    else select(prefill_select_r<32, false, kPrefSelThreads>);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark_phase(ev, SPLA_PHASE_SELECT, true, st);
  // 5. the fused pass of every group of positions
  mark_phase(ev, SPLA_PHASE_SPARSE, false, st);
  GroupArgs a;
  a.m = m;
  a.T = T;
  a.n_blk = n_blk;
  a.P = prefill_positions(m, T);
  a.n_split = prefill_splits(m, T);
  a.gw = prefill_wg_groups(a.n_split);
  a.n_grp = prefill_groups(T, a.gw * a.P);
  a.n_items = m.bh * a.n_grp * (a.n_split * a.gw / 4);
  a.stride = ws.part_stride;
  a.s = cfg.softmax_scale > 0.f ? cfg.softmax_scale : (float)(1.0 / sqrt((double)m.d));
  a.eps = cfg.rms_eps;
  a.flags = cfg.flags;
  a.kc = (const bf16_t*)c.k_cache;
  a.vc = (const bf16_t*)c.v_cache;
  a.q = q;
  a.seq_lens = c.seq_lens;
  a.sel = (const int32_t*)(base + ws.sel);
  a.table = m.pages > 0 ? c.block_table : nullptr;
  a.s_hi = (const uint4*)(base + ws.s_hi);
  a.s_lo = (const uint4*)(base + ws.s_lo);
  a.z_pre = (const float*)(base + ws.z_pre);
  a.gamma = gamma;
  a.part = (float*)(base + ws.part);
  a.out = out;
  if (m.B == 32) prefill_group_db<D, 32>(a, st);
  else if (m.B == 64) prefill_group_db<D, 64>(a, st);
  else prefill_group_db<D, 128>(a, st);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark_phase(ev, SPLA_PHASE_SPARSE, true, st);
  // 6. split groups: records, residual, RMSNorm, outputs
  mark_phase(ev, SPLA_PHASE_MERGE, false, st);
  if (a.n_split > 1)
    hipLaunchKernelGGL((prefill_merge_kernel<D>), dim3((unsigned)((int64_t)m.bh * T)),
                       dim3(64 * m.group), 0, st, m, T, cfg.rms_eps, cfg.flags, gamma,
                       (const int32_t*)c.seq_lens, (const float*)(base + ws.part), a.n_split,
                       ws.part_stride, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  mark_phase(ev, SPLA_PHASE_MERGE, true, st);
  // 7. the sequences' lengths
  return launch_append_finish(m, c, T, nullptr, st);
}

hipError_t launch_prefill_chunk(const Dims& m, const spla_config& cfg, const spla_cache& c,
                                int T, const void* k_new, const void* v_new, const void* q,
                                const float* gamma, void* out, int32_t* sel_out,
                                const PrefillWs& ws, char* base, const spla_events* ev,
                                hipStream_t st) {
  if (T < 1 || T > ws.T) return hipErrorInvalidValue;
  auto run = m.d == 64 ? prefill_chunk_d<64> : prefill_chunk_d<128>;
  return run(m, cfg, c, T, (const bf16_t*)k_new, (const bf16_t*)v_new, (const bf16_t*)q, gamma,
             (bf16_t*)out, sel_out, ws, base, ev, st);
}

}  // namespace spla
