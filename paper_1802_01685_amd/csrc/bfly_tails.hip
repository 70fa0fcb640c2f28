// Single-pass kappa-sigma tail search (Sec. 2.2 and the Fig. 5 caption: sigma is predicted by
// Parseval's theorem, and only correlations above kappa sigma leave the GPU).
//
// sigma_k^2 = (1/n_ok) sum_tau rho_k(tau)^2 is complete only after every offset, so an exact
// tail extraction needs sigma before the pass that forms rho.  The predictor here takes the
// paper's route in the lag domain: with z the series normalised window by window (centred
// and scaled by 1/sqrt(E) of the window around each sample), sum_tau (h . z_tau)^2 equals
// sum_l R_h(l) R_z(l) over the lags |l| < L, R the autocorrelations, which by Parseval is
// sum_f |H(f)|^2 Q(f) / N with Q the cosine transform of R_z.  The search pass then keeps
// every (tau, k) with |rho| above kappa * margin * sigma_pred as a candidate (the FFT form:
// every (block, k) pair holding one) while it sums the exact rho^2; afterwards the exact
// thresholds kappa * sigma_k select the tails among the candidates (the FFT form transforms
// the listed pairs again).  That is exact whenever no exact threshold lies below its
// predicted one and the candidates fit.  Templates for which the first fails are handled by
// themselves: the FFT form lists all their blocks for the second transform, the direct forms
// run the ordinary tails pass over the template tiles that hold one; a series whose candidates
// did not fit gets the whole pass, and so does an FFT batch that lists most of its pairs.  Either
// way the tails, sigma and counts are those of the two-pass search, bit for bit.
#include "bfly_internal.h"

#include <hip/hip_runtime.h>

namespace bfly {

namespace {

// z[j] = (x[j] - mean of the window around j) / sqrt(E of that window), the window around j
// being tau = clamp(j - L/2, 0, W - 1); 0 where that window is degenerate or x[j] is not
// finite.
__global__ __launch_bounds__(256) void k_zloc(const BatchHdr* __restrict__ hdr, int L) {
  if ((int)blockIdx.y >= hdr->n_segs) return;
  const SegDesc& sg = hdr_segs(hdr)[blockIdx.y];
  if (!sg.zloc) return;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) sg.acf[L] = 0.0;   // k_acf_sum counts into it
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < sg.n; j += stride) {
    int64_t tau = j - L / 2;
    tau = tau < 0 ? 0 : (tau >= sg.W ? sg.W - 1 : tau);
    const double s = sg.inv_norm[tau];
    float z = 0.0f;
    const float v = sg.x[j];
    if (s > 0.0 && isfinite(v)) {
      // the window mean of x from the prefix sums (the level cancels)
      const double s1 = (sg.pre[4 * (tau + L)] - sg.pre[4 * tau]) +
                        (sg.pre[4 * (tau + L) + 1] - sg.pre[4 * tau + 1]);
      z = (float)(((double)v - s1 / (double)L) * s);
    }
    sg.zloc[j] = z;
  }
}

// Lag sums over one chunk of the series: block (256 lags, chunk, series); acf_part[chunk][l] =
// sum over j in the chunk of z[j] z[j + l], in float64.  A lane takes 4 consecutive lags and,
// of every tile of samples, its wave a quarter; four samples at a time, so that 16 products
// share three 16-byte LDS reads (one product per two reads took 122 us for two series of
// 65,536 samples at L = 4096; this 45 us).  The four waves' sums are added in a fixed order
// (deterministic).
constexpr int ACF_TILE = 1024;
constexpr int ACF_LAGS = 256;
__global__ __launch_bounds__(256) void k_acf(const BatchHdr* __restrict__ hdr, int L) {
  if ((int)blockIdx.z >= hdr->n_segs) return;
  const SegDesc& sg = hdr_segs(hdr)[blockIdx.z];
  if (!sg.zloc) return;
  __shared__ float4 zj4[ACF_TILE / 4];
  __shared__ float4 zt4[(ACF_TILE + ACF_LAGS) / 4];
  __shared__ double part[4][ACF_LAGS];
  float* zj = (float*)zj4;
  float* zt = (float*)zt4;
  const int t = threadIdx.x, lane = t & 63, ph = t >> 6;
  const int64_t n = sg.n;
  const int64_t per = (n + ACF_CHUNKS - 1) / ACF_CHUNKS;
  const int64_t j_lo = (int64_t)blockIdx.y * per;
  const int64_t j_hi = j_lo + per < n ? j_lo + per : n;
  const int l0 = (int)blockIdx.x * ACF_LAGS;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t j0 = j_lo; j0 < j_hi; j0 += ACF_TILE) {
    __syncthreads();
    // zj[i] = z[j0 + i] within the chunk, zt[i] = z[j0 + l0 + i]; both 0 outside, which adds
    // nothing to a sum
    for (int i = t; i < ACF_TILE + ACF_LAGS; i += 256) {
      const int64_t jj = j0 + l0 + i;
      zt[i] = jj < n ? sg.zloc[jj] : 0.0f;
    }
    for (int i = t; i < ACF_TILE; i += 256) {
      const int64_t jj = j0 + i;
      zj[i] = jj < j_hi ? sg.zloc[jj] : 0.0f;
    }
    __syncthreads();
    for (int q = ph * (ACF_TILE / 16); q < (ph + 1) * (ACF_TILE / 16); ++q) {
      const float4 s = zj4[q], u = zt4[q + lane], v = zt4[q + lane + 1];
      const double a[4] = {s.x, s.y, s.z, s.w};
      const double w[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
      for (int l = 0; l < 4; ++l)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[l] = fma(a[i], w[i + l], acc[l]);
    }
  }
#pragma unroll
  for (int l = 0; l < 4; ++l) part[ph][4 * lane + l] = acc[l];
  __syncthreads();
  if (l0 + t < L)
    sg.acf_part[(int64_t)blockIdx.y * L + l0 + t] = ((part[0][t] + part[1][t]) + part[2][t]) + part[3][t];
}

// acf[l] = sum of the chunks' lag sums in chunk order; acf[L] (0 before) += non-degenerate
// offsets (whole numbers: exact in any order).
__global__ __launch_bounds__(256) void k_acf_sum(const BatchHdr* __restrict__ hdr, int L) {
  if ((int)blockIdx.y >= hdr->n_segs) return;
  const SegDesc& sg = hdr_segs(hdr)[blockIdx.y];
  if (!sg.zloc) return;
  const int l = (int)blockIdx.x * 256 + threadIdx.x;
  if (l < L) {
    double a = 0.0;
    for (int c = 0; c < ACF_CHUNKS; ++c) a += sg.acf_part[(int64_t)c * L + l];
    sg.acf[l] = a;
  }
  int mine = 0;
  for (int64_t tau = l; tau < sg.W; tau += (int64_t)gridDim.x * 256)
    mine += sg.inv_norm[tau] > 0.0 ? 1 : 0;
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) mine += __shfl_xor(mine, o, 64);
  if ((threadIdx.x & 63) == 0 && mine) atomicAdd(sg.acf + L, (double)mine);
}

// Q(f) = R(0) + 2 sum_{l=1}^{L-1} R(l) cos(2 pi f l / N), f = 0 .. N/2, N a power of two.  A
// block takes 64 frequencies at a time, one per lane, and each of its 16 waves a sixteenth of the
// lags (one thread per frequency over all lags took 175 us at L = 4096; this 27 us).  With many
// series a block takes more frequencies, up to all of a series (launch_qspec): with a table for
// every 64 frequencies 1,000 series of L = 600 took 2.0 ms and 4,000 of L = 64 5.0, this 0.96 and
// 0.80.
constexpr int QSPEC_WAVES = 16;
__global__ __launch_bounds__(1024) void k_qspec(const BatchHdr* __restrict__ hdr, int L, int N) {
  if ((int)blockIdx.y >= hdr->n_segs) return;
  const SegDesc& sg = hdr_segs(hdr)[blockIdx.y];
  if (!sg.zloc) return;
  __shared__ float ct[8192];
  __shared__ double rl[MAX_L];   // R(0), 2 R(1), 2 R(2), ...
  __shared__ double part[QSPEC_WAVES][64];
  for (int i = threadIdx.x; i < N; i += 1024) {
    double sn, cs;
    sincospi(2.0 * (double)i / (double)N, &sn, &cs);
    ct[i] = (float)cs;
  }
  for (int l = threadIdx.x; l < L; l += 1024) rl[l] = l ? 2.0 * sg.acf[l] : sg.acf[0];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lmax = L < N ? L : N;
  const int per = (lmax + QSPEC_WAVES - 1) / QSPEC_WAVES;
  const int hi = (wave + 1) * per < lmax ? (wave + 1) * per : lmax;
  for (int f0 = (int)blockIdx.x * 64; f0 <= N / 2; f0 += (int)gridDim.x * 64) {
    const int f = f0 + lane;
    double q = 0.0;
    for (int l = wave * per; l < hi; ++l)
      q = fma(rl[l], (double)ct[(f * l) & (N - 1)], q);
    part[wave][lane] = q;
    __syncthreads();
    if (wave == 0 && f <= N / 2) {
      double s = 0.0;
      for (int w = 0; w < QSPEC_WAVES; ++w) s += part[w][lane];
      sg.qspec[f] = (float)s;
    }
    __syncthreads();   // the next frequencies overwrite the sums
  }
}

__device__ __forceinline__ void flag_all(BatchHdr* hdr, const SegDesc& sg) {
  atomicOr(sg.redo, REDO_ALL);
  hdr->redo_any = 1u;
}

// Per series: REDO_ALL if the candidates of a shard did not fit; direct forms: REDO_TILES if an
// exact threshold lies below its predicted lower one, with the first bound of each such tile
// of TILE_K templates overwritten by -1 (bounds are not negative).  One wave per tile.
__global__ __launch_bounds__(256) void k_tails_check(BatchHdr* __restrict__ hdr, BankDev b) {
  if ((int)blockIdx.y >= hdr->n_segs) return;
  const SegDesc& sg = hdr_segs(hdr)[blockIdx.y];
  if (!sg.redo) return;
  const int64_t per = sg.cand_cap / CAND_SHARDS;
  if (blockIdx.x == 0 && threadIdx.x < CAND_SHARDS && (int64_t)sg.n_cand[threadIdx.x] > per)
    flag_all(hdr, sg);
  if (b.precision == P_FFT) {   // k_fft_pair_list has listed those templates' blocks
    static_assert(CAND_SHARDS == 256, "one thread per shard");
    if (blockIdx.x == 0) {
      unsigned long long n = sg.n_cand[threadIdx.x];
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) n += __shfl_xor(n, o, 64);
      if ((threadIdx.x & 63) == 0 && n) atomicAdd(&hdr->listed, n);
    }
    return;
  }
  static_assert(TILE_K == WAVE, "one lane per template of a tile");
  const int lane = threadIdx.x & 63;
  const int64_t n_tiles = b.K_pad / TILE_K;
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < n_tiles;
       t += (int64_t)gridDim.x * 4) {
    const int64_t k = t * TILE_K + lane;
    const bool bad = k < b.K && !(sg.thr[k] >= sg.thr_lo[k]);
    if (__any(bad) && lane == 0) {
      sg.thr_lo[t * TILE_K] = -1.0f;
      atomicOr(sg.redo, REDO_TILES);
    }
  }
}

// Every candidate above its exact threshold is a tail, unless the tails pass takes the series
// or the candidate's tile.
__global__ __launch_bounds__(256) void k_tails_keep(const BatchHdr* __restrict__ hdr, BankDev b) {
  if ((int)blockIdx.y >= hdr->n_segs) return;
  const SegDesc& sg = hdr_segs(hdr)[blockIdx.y];
  if (!sg.redo || (sg.redo[0] & REDO_ALL)) return;
  const bool tiles = sg.redo[0] != 0u;
  const int64_t per = sg.cand_cap / CAND_SHARDS;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < per * CAND_SHARDS;
       i += stride) {
    if ((unsigned long long)(i % per) >= sg.n_cand[i / per]) continue;
    const int32_t kl = sg.c_k[i];
    const float rf = sg.c_rho[i];
    if (fabsf(rf) > sg.thr[kl] && !(tiles && sg.thr_lo[kl & ~(TILE_K - 1)] < 0.0f)) {
      const unsigned long long slot = atomicAdd(sg.n_tails, 1ull);
      if ((int64_t)slot < sg.tail_cap) {
        sg.t_tau[slot] = sg.c_tau[i];
        sg.t_k[slot] = (int32_t)(b.k_offset + kl);
        sg.t_rho[slot] = rf;
      }
      atomicAdd(sg.t_bins + kl / b.n_fdot, 1u);
    }
  }
}

}  // namespace

int pred_points(const BankDev& b) {
  if (b.precision == P_FFT) return 2 * b.fft_m;
  int n = 1024;
  while (n < 2 * b.L - 1 && n < 8192) n *= 2;
  return n;
}

hipError_t launch_acf(const BatchHdr* hdr, int32_t seg_slots, int L, hipStream_t s) {
  hipLaunchKernelGGL(k_zloc, dim3(256, (unsigned)seg_slots), dim3(256), 0, s, hdr, L);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_acf, dim3((unsigned)((L + ACF_LAGS - 1) / ACF_LAGS), ACF_CHUNKS, (unsigned)seg_slots),
                     dim3(256), 0, s, hdr, L);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_acf_sum, dim3((unsigned)((L + 255) / 256), (unsigned)seg_slots),
                     dim3(256), 0, s, hdr, L);
  return hipGetLastError();
}

hipError_t launch_qspec(const BatchHdr* hdr, int32_t seg_slots, int L, int pred_n,
                        hipStream_t s) {
  const int groups = (pred_n / 2 + 1 + 63) / 64;
  // groups of 64 frequencies per block: the fewest rounds of 256 blocks (one per CU) times a
  // block's time, 5 us for its table and 0.35 + 0.0054 L us per group, in units of the last
  int xb = groups;
  int64_t best = INT64_MAX;
  for (int x = groups; x >= 1; --x) {
    const int64_t rounds = ((int64_t)x * seg_slots + 255) / 256;
    const int64_t cost = rounds * ((groups + x - 1) / x * (int64_t)(L + 65) + 925);
    if (cost < best) {
      best = cost;
      xb = x;
    }
  }
  hipLaunchKernelGGL(k_qspec, dim3((unsigned)xb, (unsigned)seg_slots), dim3(64 * QSPEC_WAVES), 0, s,
                     hdr, L, pred_n);
  return hipGetLastError();
}

hipError_t launch_tails_check(BatchHdr* hdr, int32_t seg_slots, const BankDev& b,
                              hipStream_t s) {
  const int64_t xb = (b.K_pad + 255) / 256;
  hipLaunchKernelGGL(k_tails_check, dim3((unsigned)(xb < 1024 ? (xb > 0 ? xb : 1) : 1024), (unsigned)seg_slots),
                     dim3(256), 0, s, hdr, b);
  return hipGetLastError();
}

hipError_t launch_tails_keep(const BatchHdr* hdr, int32_t seg_slots, const BankDev& b,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_tails_keep, dim3(256, (unsigned)seg_slots), dim3(256), 0, s, hdr, b);
  return hipGetLastError();
}

}  // namespace bfly
