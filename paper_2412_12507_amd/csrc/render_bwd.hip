// K6 + K7 -- backward of the compositing and of the per-particle colour
// (Supp. B).  No gradient flows through the sigma-point projection, the
// rectangles or the sort order (Sec. 4.1: the UT only selects particles).
//
// K6 (per tile, same layout as the forward): each pixel recomputes its
// contributors front to back with the forward's exact arithmetic, up to its
// stored n_contrib.  For contributor j with transmittance T_j before it,
//   dL/dalpha_j = sum_ch gC (c_j T_j - (S_after + T_N bg) / (1 - alpha_j))
//                 - gT T_N / (1 - alpha_j),   S_after = C - T_N bg - C_<=j,
//   dL/dc_j     = alpha_j T_j gC,
// and through alpha = sigma exp(-omega^2/2) (unclamped only):
//   dL/dsigma += dL/dalpha exp(-omega^2/2),
//   dL/domega^2 = -alpha/2 dL/dalpha.
// With p = o_g + tau d_g = (d_g x (o_g x d_g)) / |d_g|^2 the closest point
// in canonical space, d omega^2/d o_g = 2p and d omega^2/d d_g = 2 tau p
// (Supp. B), so with M = S^-1 R^T the per-pixel gradients are
//   dL/dmu = -M^T c p,   dL/dM = c p (M^-1 p)^T,   c = 2 dL/domega^2.
// They only depend on G = sum c p p^T (6 values) and h = sum c p (3): those
// plus dL/dsigma and dL/dc are summed over the pixels of a 4 x 4 block in FP32
// (one reduce-scatter for all 13), over the tile in FP64 in LDS, and over the
// tiles by one FP64 atomic per value and (tile, particle), so the
// per-particle totals carry no order-dependent FP32 rounding.  (By pairs: over two
// such blocks in FP32, over the half tile in FP64, one atomic per value and
// (half tile, particle).)
//
// K7 (per particle) then applies M = S^-1 R^T:
//   dL/ds_k = -G_kk / s_k,   dL/dR = R S G S^-1,   dL/dmu = -R S^-1 h,
// the quaternion normalisation Jacobian, and (per camera) the SH colour:
//   dL/dbeta_k = dL/dc Y_k(d),  dL/dmu += (I - d d^T)/|mu - o| sum beta grad Y.
#include <mutex>

#include "camera_dev.h"
#include "tile_eval.h"

namespace gut {

constexpr int kAcc = 10;  // G xx,xy,xz,yy,yz,zz ; h x,y,z ; dL/dsigma

// Sums 16 per-lane values over each row of 16 lanes as a reduce-scatter (DPP
// only): at each step a lane keeps half of its values and adds its partner's
// copy of that half.  Lane l then holds its row's total of value l mod 16.
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_reduce16(const float (&g)[16], int lane) {
  float h8[8], h4[4], h2[2];
  const bool b3 = lane & 8, b2 = lane & 4, b1 = lane & 2, b0 = lane & 1;
#pragma unroll
  for (int j = 0; j < 8; j++)  // partner lane ^ 8 (row rotate by 8)
    h8[j] = (b3 ? g[j + 8] : g[j]) + dpp<0x128>(b3 ? g[j] : g[j + 8]);
#pragma unroll
  for (int j = 0; j < 4; j++)  // partner 7 - (lane mod 8) (row half-mirror): differs in bit 2
    h4[j] = (b2 ? h8[j + 4] : h8[j]) + dpp<0x141>(b2 ? h8[j] : h8[j + 4]);
#pragma unroll
  for (int j = 0; j < 2; j++)  // partner 3 - (lane mod 4) (quad mirror): differs in bit 1
    h2[j] = (b1 ? h4[j + 2] : h4[j]) + dpp<0x1B>(b1 ? h4[j] : h4[j + 2]);
  return (b0 ? h2[1] : h2[0]) + dpp<0xB1>(b0 ? h2[0] : h2[1]);  // partner lane ^ 1
}

constexpr int kBwThreads = 256;
constexpr int kBwBatch = 128;  // pairs of 192 bytes: three blocks a CU, as many waves as the registers allow
constexpr int kRow = kAcc + 3;  // sums per pair

// A thread's pixel.  Its contributors lie before list position `last` (0:
// none, or outside the image).  T and Z run along the list: the transmittance,
// and Z = sum_c gC_c (C_c - C_<=j,c) in FP64 (C the output colour, C_<=j the
// running colour including entry j), which is all the suffix sums S_after
// enter the gradient through; gTT = T_N gT.
struct BwPixel {
  float u, v, dt, dlen, clip, T, gC[3], gTT;
  double Z;
  uint32_t last;
};

__device__ __forceinline__ bool finite3(const float (&x)[3]) {
  return fabsf(x[0]) < INFINITY && fabsf(x[1]) < INFINITY && fabsf(x[2]) < INFINITY;
}

// A pixel's terms of one entry: the closest point q, c q, the factor of rho in
// dL/dsigma and the weight of the loss gradient in dL/dc.
struct BwTerms {
  float3 q, cq;
  float s, w;
};

// Blends the entry (colour cold) on a pixel it hits, and its terms, zero but for
// q on a pixel that is not hit.
template <bool RS, bool GEN>
__device__ __forceinline__ void bwd_terms(const PairRegs<RS>& r, const float4* P, const double (&cold)[3],
                                          const Thresholds& th, bool hit, Eval& ev, BwPixel& p, BwTerms& o) {
  eval_alpha<RS, GEN>(r, th, &ev);
  const float Tb = p.T;
  const float ae = hit ? ev.a : 0.0f;
  o.w = ae * Tb;
  p.T = fmaf(-ae, Tb, Tb);  // the forward's update, bit for bit
  // D = gC . c_j; after this entry Z = sum_c gC_c (C_c - C_<=j,c)
  const double D = fma((double)p.gC[0], cold[0], fma((double)p.gC[1], cold[1], (double)p.gC[2] * cold[2]));
  p.Z = fma(-(double)o.w, D, p.Z);
  // dL/dalpha = T_j gC.c_j - (gC.(C - C_<=j) + gT T_N) / (1 - alpha_j)
  const float inv1m = __builtin_amdgcn_rcpf(1.0f - ev.a);
  float gA = fmaf(Tb, (float)D, -inv1m * ((float)p.Z + p.gTT));
  const bool geo = hit && !ev.clamped;  // alpha = alpha_max carries no gradient
  gA = geo ? gA : 0.0f;
  // 2 dL/domega^2; a degree-n response scales d alpha / d omega^2 by
  // 2 lambda (n/2) (omega^2)^(n/2 - 1) relative to the Gaussian's
  // (0 for a lane that is not hit, whose omega may be infinite)
  float c = -ev.a * gA;
  if (GEN) c = geo ? c * __builtin_amdgcn_exp2f(fmaf(th.k_h - 1.0f, ev.lq, th.k_f)) : 0.0f;
  float3 dg, cr;
  pair_vectors<RS>(P, ev, p.u, p.v, &dg, &cr);
  const float3 q = cross3f_fma(dg, cr);
  o.q = f3(q.x * ev.idd, q.y * ev.idd, q.z * ev.idd);
  o.cq = f3(c * o.q.x, c * o.q.y, c * o.q.z);
  o.s = gA * (ev.araw * __builtin_amdgcn_exp2f(-r.lsig));  // rho = (sigma rho) / sigma
}

// One step: each lane's own list entry (at list position idx) against its
// pixel: the pixel's terms of the entry's sums, G = sum c p p^T (symmetric,
// 6), h = sum c p (3), dL/dsigma, dL/dc (3), zero where it is not hit.
// Returns false when no lane is hit (g is then not written).  odd (uniform over
// the wave): the loss gradient of some pixel is not finite.
template <bool RS, bool GEN, bool CLIP>
__device__ __forceinline__ bool bwd_step(const PairRegs<RS>& r, const float4* P, uint32_t idx, bool mixed, bool odd,
                                         const Thresholds& th, BwPixel& p, float (&g)[16]) {
  Eval ev;
  eval_test<RS>(r, P, p.u, p.v, p.dt, mixed, &ev);
  if (CLIP) clip_test<RS>(r, P, p.u, p.v, p.dt, p.dlen, p.clip, &ev);
  const bool in = idx < p.last, on = eval_hit<RS>(r, ev);
  if ((__builtin_amdgcn_ballot_w64(on) & __builtin_amdgcn_ballot_w64(in)) == 0ull) return false;
  const bool hit = on && in;
  double cold[3];
  pair_colour<RS>(P, cold);
  BwTerms o;
  bwd_terms<RS, GEN>(r, P, cold, th, hit, ev, p, o);
  g[0] = o.cq.x * o.q.x;
  g[1] = o.cq.x * o.q.y;
  g[2] = o.cq.x * o.q.z;
  g[3] = o.cq.y * o.q.y;
  g[4] = o.cq.y * o.q.z;
  g[5] = o.cq.z * o.q.z;
  g[6] = o.cq.x;
  g[7] = o.cq.y;
  g[8] = o.cq.z;
  g[9] = o.s;
  g[10] = o.w * p.gC[0];
  g[11] = o.w * p.gC[1];
  g[12] = o.w * p.gC[2];
  // An infinite or NaN gradient does not reach entries its pixel does not blend.
  // (As selects in every step this takes 0.8% of a 1M fisheye training step,
  // behind a branch nothing; of a rolling one, whose longest tiles wait for each
  // step, the branch takes 1% and selects 0.3%.)
  if (RS || odd) {
    if (!RS) asm volatile("");  // (kept a branch)
    g[10] = hit ? g[10] : 0.0f;
    g[11] = hit ? g[11] : 0.0f;
    g[12] = hit ? g[12] : 0.0f;
  }
  g[13] = g[14] = g[15] = 0.0f;
  return true;
}

// The step on pair i of the batch from list position b on, and its sums into
// the pair's row (of the lists' padding too, kChunk, whose sums are zero).
static_assert(kChunk <= kBwBatch, "the padding has a row");
template <bool RS, bool GEN, bool CLIP>
__device__ __forceinline__ void bwd_pair(const PairRegs<RS>& r, const float4* pd, uint32_t i, uint32_t b, bool mixed,
                                         bool odd, const Thresholds& th, BwPixel& p, double* rows, int lane) {
  float g[16];
  if (!bwd_step<RS, GEN, CLIP>(r, pd + i * Slots<RS, true>::N, b + i, mixed, odd, th, p, g)) return;
  const float tot = row_reduce16(g, lane);
  if ((lane & 15) < kRow && tot != 0.0f) atomicAdd(&rows[i * kRow + (lane & 15)], (double)tot);
}

// Adds the batch's rows to the per-particle sums and clears them: 16 lanes per
// row, so that a particle's values go out together.
__device__ inline void bwd_flush(double* rows, const uint32_t* pe, int m, int n, int cam_idx,
                                 double* __restrict__ acc, double* __restrict__ acc_rgb) {
  const int k = threadIdx.x & 15;
  if (k >= kRow) return;
  for (int r = threadIdx.x >> 4; r < m; r += kBwThreads / 16) {
    const double x = rows[r * kRow + k];
    if (x == 0.0) continue;
    rows[r * kRow + k] = 0.0;
    const uint32_t e = pe[r];
    const long long i = (long long)(e - (uint32_t)cam_idx * (uint32_t)n);
    if (k < kAcc) atomicAdd(&acc[i * kAcc + k], x);
    else atomicAdd(&acc_rgb[3 * (long long)e + (k - kAcc)], x);
  }
}

// The forward's blocks, pixels, pair setup and lists (NQ = 1).  A step sums its pixels'
// terms over each row of lanes (up to four different pairs at once) and adds
// the rows' totals to the pairs' rows in LDS, in FP64; a row goes to the
// per-particle sums when its batch is done, one atomic per value and (tile,
// particle).  Three waves a SIMD do not hide a step's chain of LDS reads (the
// place in the list, then the pair), so both are read ahead of the step that
// uses them: a training step of 1M particles at 1920x1080 1400 -> 1342 us, of
// 300k with a rolling shutter at 800x600 1181 -> 1067 us.
template <bool RS, bool GEN, bool CLIP>
__global__ void __launch_bounds__(kBwThreads, 3) render_bwd_kernel(
    DevCam cam, Thresholds th, int n, int cam_idx, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ ids,
    const float4* __restrict__ record, const float* __restrict__ clip,
    const float* __restrict__ rgb, const float* __restrict__ out_rgb,
    const float* __restrict__ out_T, const uint32_t* __restrict__ out_nc,
    const float* __restrict__ d_rgb, const float* __restrict__ d_T, double* __restrict__ acc,
    double* __restrict__ acc_rgb) {
  constexpr int S = Slots<RS, true>::N;
  __shared__ float4 pd[batch_rows(kBwBatch) * S];
  __shared__ double rows[(kBwBatch + 1) * kRow];  // the last one the padding's, never read
  __shared__ uint32_t pe[2][kBwBatch];  // the entries of this batch and of the one before
  __shared__ unsigned short pf[kBwBatch];
  __shared__ WaveLists lists[kBwThreads / 64];
  __shared__ TileFrameD F;
  __shared__ QuadBoxes wb;
  __shared__ float red[12];
  __shared__ uint32_t maxlast_s;

  const int tile = (int)order[cam.tile_base + blockIdx.x];  // longest lists first
  const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
  const int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  int px, py;
  lane_pixel(wv, lane, &px, &py);
  px += tx * kTile;
  py += ty * kTile;
  if (t == 0) { tile_frame(cam, tx, ty, &F); maxlast_s = 0; }
  // the padding's row (written for any number of chunks and threads: with the
  // bounds as constants the compiler makes the whole kernel 2% slower under a
  // rolling shutter, 558 against 548 us for 300k particles at 800x600)
  for (int i = t; i < (kBwBatch + kChunk - 1) / kChunk * S; i += blockDim.x)
    pd[((i / S + 1) * (kChunk + 1) - 1) * S + i % S] = dummy_slot<RS>(i % S);
  for (int i = t; i < (kBwBatch + 1) * kRow; i += kBwThreads) rows[i] = 0.0;
  __syncthreads();

  BwPixel p = {};
  const bool active = px < cam.W && py < cam.H && pixel_ray(cam, F, px, py, &p.u, &p.v, &p.dt);
  float umax, vmax, dtmax;
  tile_bounds<1>(&p.u, &p.v, &p.dt, &active, red, &umax, &vmax, &dtmax);
  const float l2amin = log2f(th.alpha_min);
  const BlockBox box = block_box(p.u, p.v, active, 5e-7f * (umax + vmax), wv, &wb);
  const long long pix = cam.pixel_base + (long long)py * cam.W + px;
  if (CLIP) {  // the forward's clip test operands
    if (active) {
      p.clip = clip[pix];
      p.dlen = sqrtf(fmaf(p.u, p.u, fmaf(p.v, p.v, 1.0f)));
    }
    quad_clip_max(p.clip, active, wv, &wb);
  }
  p.T = 1.0f;
  if (active) {
    p.last = out_nc[pix];
    p.gTT = (d_T ? d_T[pix] : 0.0f) * out_T[pix];
    for (int c = 0; c < 3; c++) {
      p.gC[c] = d_rgb[3 * pix + c];
      p.Z = fma((double)p.gC[c], (double)out_rgb[3 * pix + c], p.Z);
    }
  }
  const bool odd = wave_any(!finite3(p.gC));
  atomicMax(&maxlast_s, p.last);
  __syncthreads();  // (also publishes wb)
  const uint2 rg = ranges[cam.tile_base + tile];
  // never past the tile's list
  const uint32_t maxlast = __builtin_amdgcn_readfirstlane(min(maxlast_s, rg.y - rg.x));
  if (maxlast >= 2048) __builtin_amdgcn_s_setprio(3);
  else if (maxlast >= 1024) __builtin_amdgcn_s_setprio(2);
  else if (maxlast >= 256) __builtin_amdgcn_s_setprio(1);

  int par = 0, m = 0;  // pairs of the batch in rows
  for (uint32_t b = 0; b < maxlast; b += kBwBatch) {
    if (b) {
      __syncthreads();
      bwd_flush(rows, pe[par], m, n, cam_idx, acc, acc_rgb);
      par ^= 1;
    }
    m = (int)min(maxlast - b, (uint32_t)kBwBatch);
    if (t < kBwBatch) {
      uint32_t fl = 0u;
      if (t < m) {
        const uint32_t e = ids[rg.x + b + t];
        pe[par][t] = e;
        fl = pair_setup<RS, true, GEN, CLIP>(record, rgb, e, (int)(e - (uint32_t)cam_idx * (uint32_t)n), F,
                                             cam, umax, vmax, dtmax, th, l2amin, wb, &pd[t * S]);
      }
      pf[t] = (unsigned short)fl;
    }
    __syncthreads();
    if (!wave_any(b < p.last)) continue;
    // (the blocks' pixels that still have contributors: a subset of the forward's)
    const uint32_t lm = build_lists<RS, true>(pd, pf, wv, box, b < p.last, lists[wv]);
    const int cnt = (int)(lm & ~kMixed);
    const bool mixed = (lm & kMixed) != 0u;
    const unsigned char* mine = lists[wv].row[lane >> 4];
    if (cnt == 0) continue;
    // places are read two steps ahead and pairs one (the lists end in a few dummies)
    uint32_t i0 = mine[0], i1 = mine[1];
    PairRegs<RS> r0, r1;
    load_pair<RS>(pd + i0 * S, r0);
    for (int k = 0; k < cnt; k += 2) {
      load_pair<RS>(pd + i1 * S, r1);
      const uint32_t i2 = mine[k + 2];
      bwd_pair<RS, GEN, CLIP>(r0, pd, i0, b, mixed, odd, th, p, rows, lane);
      i0 = i2;
      load_pair<RS>(pd + i0 * S, r0);
      const uint32_t i3 = mine[k + 3];
      bwd_pair<RS, GEN, CLIP>(r1, pd, i1, b, mixed, odd, th, p, rows, lane);
      i1 = i3;
    }
  }
  __syncthreads();
  bwd_flush(rows, pe[par], m, n, cam_idx, acc, acc_rgb);
}

// The same by pairs: 128 threads, a wave for two quadrants and a thread for a
// pixel of either, as the forward's pair walk.  A step takes one pair against
// both pixels of each lane, whose terms are added before the sum over each row
// of lanes (so 32 pixels are summed in FP32); the rows' totals are added in
// FP64 and go to the per-particle sums, one atomic per value and (wave,
// particle).  See bwd_by_pairs for where this wins.
constexpr int kBpThreads = 128, kBpBatch = 128;

// x summed over the wave's four rows of 16 lanes, in every row.
__device__ __forceinline__ double rows_sum(double x) {
  uint32_t lo = (uint32_t)__double2loint(x), hi = (uint32_t)__double2hiint(x);
  auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
  auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
  x = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  lo = (uint32_t)__double2loint(x);
  hi = (uint32_t)__double2hiint(x);
  l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
  h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}

template <bool RS, bool GEN, bool CLIP>
__global__ void __launch_bounds__(kBpThreads, 3) render_bwd_pairs_kernel(
    DevCam cam, Thresholds th, int n, int cam_idx, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ ids,
    const float4* __restrict__ record, const float* __restrict__ clip,
    const float* __restrict__ rgb, const float* __restrict__ out_rgb,
    const float* __restrict__ out_T, const uint32_t* __restrict__ out_nc,
    const float* __restrict__ d_rgb, const float* __restrict__ d_T, double* __restrict__ acc,
    double* __restrict__ acc_rgb) {
  constexpr int S = Slots<RS, true>::N;
  __shared__ float4 pd[kBpBatch * S];
  __shared__ uint32_t pe[kBpBatch];
  __shared__ unsigned short pf[kBpBatch];
  __shared__ TileFrameD F;
  __shared__ QuadBoxes wb;
  __shared__ float red[6];
  __shared__ uint32_t maxlast_s;

  const int tile = (int)order[cam.tile_base + blockIdx.x];  // longest lists first
  const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
  const int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  int px, py0;  // the thread's first pixel; its second lies 8 rows below
  lane_pixel(wv, lane, &px, &py0);
  px += tx * kTile;
  py0 += ty * kTile;
  if (t == 0) { tile_frame(cam, tx, ty, &F); maxlast_s = 0; }
  __syncthreads();

  bool active[2];
  float u[2], v[2], dt[2];
#pragma unroll
  for (int k = 0; k < 2; k++) {
    u[k] = v[k] = dt[k] = 0.0f;
    active[k] = px < cam.W && py0 + 8 * k < cam.H && pixel_ray(cam, F, px, py0 + 8 * k, &u[k], &v[k], &dt[k]);
  }
  float umax, vmax, dtmax;
  tile_bounds<2>(u, v, dt, active, red, &umax, &vmax, &dtmax);
  const float l2amin = log2f(th.alpha_min);
  BwPixel p[2];
  bool odd = false;
#pragma unroll
  for (int k = 0; k < 2; k++) {
    (void)block_box(u[k], v[k], active[k], 0.0f, wv + 2 * k, &wb);
    p[k] = BwPixel{u[k], v[k], dt[k], 1.0f, 0.0f, 1.0f, {0.0f, 0.0f, 0.0f}, 0.0f, 0.0, 0u};
    const long long pix = cam.pixel_base + (long long)(py0 + 8 * k) * cam.W + px;
    if (CLIP) {  // the forward's clip test operands
      if (active[k]) {
        p[k].clip = clip[pix];
        p[k].dlen = sqrtf(fmaf(u[k], u[k], fmaf(v[k], v[k], 1.0f)));
      }
      quad_clip_max(p[k].clip, active[k], wv + 2 * k, &wb);
    }
    if (active[k]) {
      p[k].last = out_nc[pix];
      p[k].gTT = (d_T ? d_T[pix] : 0.0f) * out_T[pix];
      for (int c = 0; c < 3; c++) {
        p[k].gC[c] = d_rgb[3 * pix + c];
        p[k].Z = fma((double)p[k].gC[c], (double)out_rgb[3 * pix + c], p[k].Z);
      }
    }
    odd = odd || wave_any(!finite3(p[k].gC));
  }
  atomicMax(&maxlast_s, max(p[0].last, p[1].last));
  __syncthreads();  // (also publishes wb)
  const uint2 rg = ranges[cam.tile_base + tile];
  // never past the tile's list
  const uint32_t maxlast = __builtin_amdgcn_readfirstlane(min(maxlast_s, rg.y - rg.x));
  if (maxlast >= 2048) __builtin_amdgcn_s_setprio(3);
  else if (maxlast >= 1024) __builtin_amdgcn_s_setprio(2);
  else if (maxlast >= 256) __builtin_amdgcn_s_setprio(1);

  for (uint32_t b = 0; b < maxlast; b += kBpBatch) {
    if (b) __syncthreads();
    uint32_t fl = 0u;
    if (b + t < maxlast) {
      const uint32_t e = ids[rg.x + b + t];
      pe[t] = e;
      fl = pair_setup<RS, true, GEN, CLIP>(record, rgb, e, (int)(e - (uint32_t)cam_idx * (uint32_t)n), F, cam, umax,
                                           vmax, dtmax, th, l2amin, wb, &pd[t * S]);
    }
    pf[t] = (unsigned short)fl;
    __syncthreads();
#pragma unroll 1
    for (int h = 0; h < 2; h++) {
      // the pairs that the forward walked for the wave's quadrants
      const uint32_t f = pf[lane + 64 * h];
      unsigned long long m = __builtin_amdgcn_ballot_w64((f >> wv & 5u) != 0u);
      const unsigned long long xm = __builtin_amdgcn_ballot_w64((f & kMixedBit) != 0u);
      while (m) {
        const uint32_t ql = (uint32_t)__builtin_ctzll(m), q = 64u * h + ql, idx = b + q;
        m &= m - 1ull;
        if (!wave_any(idx < p[0].last || idx < p[1].last)) break;
        const float4* P = &pd[q * S];
        PairRegs<RS> r;
        load_pair<RS>(P, r);
        r.flag = -1.0f;  // (mixed is this pair's own)
        const uint32_t mixed = __builtin_amdgcn_readfirstlane((uint32_t)(xm >> ql) & 1u);
        Eval ev[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
          eval_test<RS>(r, P, p[k].u, p[k].v, p[k].dt, mixed != 0u, &ev[k]);
          if (CLIP) clip_test<RS>(r, P, p[k].u, p[k].v, p[k].dt, p[k].dlen, p[k].clip, &ev[k]);
        }
        const bool hit0 = eval_hit<RS>(r, ev[0]) && idx < p[0].last;
        const bool hit1 = eval_hit<RS>(r, ev[1]) && idx < p[1].last;
        if (!wave_any(hit0 || hit1)) continue;
        double cold[3];
        pair_colour<RS>(P, cold);
        BwTerms o[2];
        bwd_terms<RS, GEN>(r, P, cold, th, hit0, ev[0], p[0], o[0]);
        bwd_terms<RS, GEN>(r, P, cold, th, hit1, ev[1], p[1], o[1]);
        float g[16];
        g[0] = fmaf(o[0].cq.x, o[0].q.x, o[1].cq.x * o[1].q.x);
        g[1] = fmaf(o[0].cq.x, o[0].q.y, o[1].cq.x * o[1].q.y);
        g[2] = fmaf(o[0].cq.x, o[0].q.z, o[1].cq.x * o[1].q.z);
        g[3] = fmaf(o[0].cq.y, o[0].q.y, o[1].cq.y * o[1].q.y);
        g[4] = fmaf(o[0].cq.y, o[0].q.z, o[1].cq.y * o[1].q.z);
        g[5] = fmaf(o[0].cq.z, o[0].q.z, o[1].cq.z * o[1].q.z);
        g[6] = o[0].cq.x + o[1].cq.x;
        g[7] = o[0].cq.y + o[1].cq.y;
        g[8] = o[0].cq.z + o[1].cq.z;
        g[9] = o[0].s + o[1].s;
#pragma unroll
        for (int c = 0; c < 3; c++) g[10 + c] = fmaf(o[0].w, p[0].gC[c], o[1].w * p[1].gC[c]);
        if (odd) {  // as in bwd_step
          asm volatile("");
#pragma unroll
          for (int c = 0; c < 3; c++)
            g[10 + c] = (hit0 ? o[0].w * p[0].gC[c] : 0.0f) + (hit1 ? o[1].w * p[1].gC[c] : 0.0f);
        }
        g[13] = g[14] = g[15] = 0.0f;
        const double tot = rows_sum((double)row_reduce16(g, lane));
        if (lane < kRow && tot != 0.0) {
          const uint32_t e = pe[q];
          const long long i = (long long)(e - (uint32_t)cam_idx * (uint32_t)n);
          if (lane < kAcc) atomicAdd(&acc[i * kAcc + lane], tot);
          else atomicAdd(&acc_rgb[3 * (long long)e + (lane - kAcc)], tot);
        }
      }
    }
  }
}

// Backward of the k-buffer render ("Ours (sorted)", Sec. 4.3).  It replays
// render_kbuffer_kernel bit for bit (same blocks, pixels, pair setup, tests,
// distances, and the same buffer after every insertion: the merge chain here
// and the forward's shift-and-move for a full-size buffer order the slots
// alike, ties included) and differentiates each hit when it is blended,
// in blend order: the Supp. B recursion of render_bwd_kernel (T and
// Z = gC . (C - C_<=j) carried forward from the forward's outputs) gives
// dL/dalpha there.  The geometric factors a blend needs -- the closest-point
// vector p and rho = alpha_raw / sigma -- are formed when the hit enters the
// buffer (its pair is then in LDS) and travel with it; rho carries the sign
// of the alpha_max clamp.  The buffer alone takes 128 registers a lane; the
// kernel asks for two waves per SIMD all the same (part of it then lives in
// scratch), since the replay waits on memory far more than it computes and
// one wave per SIMD leaves the SIMD idle.
//
// Sums.  A lane blends the nearest hit of its own buffer, so the hits one
// step blends are a few different particles.  Their 13 values go to FP32 LDS
// rows by list position, over a window of the latest positions, from the last
// multiple of 256 less 256 on; a row is added to the FP64 per-particle sums
// when its batch has left the window, 13 atomics per (tile, particle).  Lanes that blend the
// same hit would meet on one LDS address, one after the other (with every
// lane adding its own values, LDS was busy 58% of the kernel, at 43 cycles an
// atomic), so each row of 16 lanes first sums the lanes that share its first
// lane's hit (the reduce-scatter of the tile-order backward) and adds the
// totals with one atomic; the lanes left over add their own.  (Going on to
// the second or fourth hit that lanes share costs more instructions than it
// saves: 1.95 and 2.08 ms a training step against 1.92.)  The
// buffer holds list positions; a hit that has stayed longer than the window
// (a buffer usually turns over within a batch) goes to the FP64 sums at once,
// each lane's values by themselves.
constexpr int kKBufB = 16;
constexpr int kKThreadsB = 256;
constexpr int kKBatchB = 128;
constexpr int kWinStep = 2 * kKBatchB;  // the window starts at a multiple of this
constexpr int kWin = 2 * kWinStep;  // list positions with an LDS row (of 13 values: an odd stride spreads them over the banks)

struct KBufGrad {
  double* acc;
  double* acc_rgb;
  const float* rgb;
  const uint32_t* lids;  // the tile's sorted entry ids
  const uint32_t* pew;   // entry ids of the window's positions (LDS)
  const float* cw;       // their colours (LDS rows of 3)
  float* accw;           // the window's rows (LDS)
  int n, cam_idx;
  float t_min;
  uint32_t wlo;  // lowest list position in the window
};

// The row of list position pos, wlo <= pos < wlo + kWin.
__device__ __forceinline__ uint32_t kbuf_row(uint32_t pos) { return pos & (kWin - 1); }

// Value k of the 13 into the FP64 sums of entry e.
__device__ __forceinline__ void kbuf_add64(uint32_t e, int k, double x, const KBufGrad& K) {
  const long long i = (long long)(e - (uint32_t)K.cam_idx * (uint32_t)K.n);
  if (k < kAcc) atomicAdd(&K.acc[i * kAcc + k], x);
  else atomicAdd(&K.acc_rgb[3 * (long long)e + (k - kAcc)], x);
}

// Adds the blended values of the lanes with act set (hit at list position
// pos) to the sums.
__device__ __forceinline__ void kbuf_add(bool act, uint32_t pos, const float (&v)[kRow], const KBufGrad& K) {
  const int lane = threadIdx.x & 63, k0 = lane & 15;
  if (__builtin_amdgcn_ballot_w64(act) == 0ull) return;
  const unsigned long long A = __builtin_amdgcn_ballot_w64(act && pos >= K.wlo);
  const uint32_t bits = (lane & 32 ? (uint32_t)(A >> 32) : (uint32_t)A) >> (lane & 16) & 0xffffu;
  const int lead = bits ? (lane & 48) + __builtin_ctz(bits) : lane;
  const uint32_t pl = (uint32_t)__shfl((int)pos, lead, 64);
  const bool match = act && pos >= K.wlo && pos == pl;
  float g[16];
#pragma unroll
  for (int k = 0; k < kRow; k++) g[k] = match ? v[k] : 0.0f;
  g[13] = g[14] = g[15] = 0.0f;
  const float tot = row_reduce16(g, lane);
  if (k0 < kRow && tot != 0.0f) atomicAdd(&K.accw[kbuf_row(pl) * kRow + k0], tot);
  act = act && !match;
  if (!act) return;
  if (pos >= K.wlo) {
    float* row = K.accw + kbuf_row(pos) * kRow;
#pragma unroll
    for (int k = 0; k < kRow; k++) atomicAdd(&row[k], v[k]);
  } else {
    const uint32_t e = K.lids[pos];
#pragma unroll
    for (int k = 0; k < kRow; k++) kbuf_add64(e, k, (double)v[k], K);
  }
}

// Adds row r of the window to the FP64 sums of its entry and clears it.
__device__ __forceinline__ void kbuf_flush_row(int r, const KBufGrad& K) {
  float* row = K.accw + r * kRow;
  const uint32_t e = K.pew[r];
#pragma unroll
  for (int k = 0; k < kRow; k++) {
    const float x = row[k];
    if (x != 0.0f) {
      kbuf_add64(e, k, (double)x, K);
      row[k] = 0.0f;
    }
  }
}

// One blend of the replay (Eq. 5 with the t_min stop, as kbuf_blend) on the
// lanes with on set, of the hit at list position pos, and its 13 gradient
// values into the sums: G (6), h (3), dL/dsigma, then dL/dc (3).  Nothing for
// a sentinel, a wall, a stopped pixel or a hit that would cross t_min.  The
// whole wave calls it.
__device__ __forceinline__ void kbuf_blend_bwd(bool on, float a, uint32_t pos, float px_, float py_, float pz_,
                                               float rho, float fg, const KBufGrad& K, const float (&gC)[3],
                                               const double (&gCd)[3], float gTT, float& T, double& Z,
                                               uint32_t& done) {
  on = on && a > 0.0f && done == 0u;
  if (!wave_any(on)) return;
  const float Tb = T;
  const float Tn = fmaf(-a, Tb, Tb);
  const bool stop = on && Tn < K.t_min;
  done = stop ? 1u : done;
  on = on && !stop;
  float v[kRow];
  if (on) {
    T = Tn;
    const float wgt = a * Tb;
    // an LDS row is read in any case and an older hit's colour then replaces
    // it; the empty register constraint keeps the compiler from folding the
    // two reads into one flat read through a selected pointer
    const float* cl = K.cw + 3 * kbuf_row(pos);
    float c0 = cl[0], c1 = cl[1], c2 = cl[2];
    asm volatile("" : "+v"(c0), "+v"(c1), "+v"(c2));
    if (pos < K.wlo) {
      const float* c = K.rgb + 3 * (size_t)K.lids[pos];
      c0 = c[0]; c1 = c[1]; c2 = c[2];
    }
    const double D = fma(gCd[0], (double)c0, fma(gCd[1], (double)c1, gCd[2] * (double)c2));
    Z = fma(-(double)wgt, D, Z);
    const float inv1m = __builtin_amdgcn_rcpf(1.0f - a);
    float gA = fmaf(Tb, (float)D, -inv1m * ((float)Z + gTT));
    if (rho < 0.0f) gA = 0.0f;  // alpha = alpha_max carries no gradient
    const float c = -a * gA * fg;  // 2 dL/domega^2 (fg: a degree-n response's chain factor, else 1)
    v[0] = c * px_ * px_; v[1] = c * px_ * py_; v[2] = c * px_ * pz_;
    v[3] = c * py_ * py_; v[4] = c * py_ * pz_; v[5] = c * pz_ * pz_;
    v[6] = c * px_; v[7] = c * py_; v[8] = c * pz_;
    v[9] = gA * fabsf(rho);
    v[10] = wgt * gC[0]; v[11] = wgt * gC[1]; v[12] = wgt * gC[2];
  }
  kbuf_add(on, pos, v, K);
}

template <bool RS, bool GEN, bool CLIP>
__global__ void __launch_bounds__(kKThreadsB, 2) render_kbuffer_bwd_kernel(
    DevCam cam, Thresholds th, int n, int cam_idx, int kcap, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ order, const uint32_t* __restrict__ ids,
    const float4* __restrict__ record, const float* __restrict__ rgb, const float* __restrict__ clip,
    const float* __restrict__ out_rgb,
    const float* __restrict__ out_T, const float* __restrict__ d_rgb, const float* __restrict__ d_T,
    double* __restrict__ acc, double* __restrict__ acc_rgb) {
  constexpr int S = Slots<RS, true>::N;
  __shared__ float4 pd[batch_rows(kKBatchB) * S];
  __shared__ unsigned short pf[kKBatchB];
  __shared__ WaveLists lists[kKThreadsB / 64];
  __shared__ uint32_t pew[kWin];
  __shared__ float cw[kWin * 3];
  __shared__ float accw[kWin * kRow];
  __shared__ TileFrameD F;
  __shared__ QuadBoxes wb;
  __shared__ float red[12];
  const int tile = (int)order[cam.tile_base + blockIdx.x];
  const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
  const int t = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  int px, py;
  lane_pixel(wv, lane, &px, &py);
  px += tx * kTile;
  py += ty * kTile;
  if (t == 0) tile_frame(cam, tx, ty, &F);
  static_assert(kKBatchB == kChunk, "one row for the padding");
  for (int i = t; i < S; i += kKThreadsB) pd[kKBatchB * S + i] = dummy_slot<RS>(i);
  for (int i = t; i < kWin * kRow; i += kKThreadsB) accw[i] = 0.0f;
  __syncthreads();
  const bool inside = px < cam.W && py < cam.H;
  float u = 0.f, v = 0.f, dt = 0.f;
  bool active = inside && pixel_ray(cam, F, px, py, &u, &v, &dt);
  float umax, vmax, dtmax;
  tile_bounds<1>(&u, &v, &dt, &active, red, &umax, &vmax, &dtmax);
  const float l2amin = log2f(th.alpha_min);
  const BlockBox box = block_box(u, v, active, 5e-7f * (umax + vmax), wv, &wb);
  const float dlen = sqrtf(fmaf(u, u, fmaf(v, v, 1.0f)));
  float clipv = 0.0f;  // the forward's clip operands
  if (CLIP) {
    if (active) clipv = clip[cam.pixel_base + (long long)py * cam.W + px];
    quad_clip_max(clipv, active, wv, &wb);
  }

  // the loss gradients and Z = gC . C_out (FP64), as in render_bwd_kernel
  float gC[3] = {0.f, 0.f, 0.f}, gTT = 0.f;
  double gCd[3] = {0.0, 0.0, 0.0}, Z = 0.0;
  if (active) {
    const long long pix = cam.pixel_base + (long long)py * cam.W + px;
    gTT = (d_T ? d_T[pix] : 0.0f) * out_T[pix];
    for (int c = 0; c < 3; c++) {
      gC[c] = d_rgb[3 * pix + c];
      gCd[c] = gC[c];
      Z = fma(gCd[c], (double)out_rgb[3 * pix + c], Z);
    }
  }
  const uint2 rg = ranges[cam.tile_base + tile];
  const uint32_t len = __builtin_amdgcn_readfirstlane(rg.y - rg.x);
  KBufGrad K = {acc, acc_rgb, rgb, ids + rg.x, pew, cw, accw, n, cam_idx, th.t_min, 0u};

  float bd[kKBufB], ba[kKBufB], bx[kKBufB], by[kKBufB], bz[kKBufB], br[kKBufB], bf[kKBufB];
  uint32_t bi[kKBufB];  // list positions
#pragma unroll
  for (int j = 0; j < kKBufB; j++) {
    bd[j] = j < kcap ? -INFINITY : INFINITY;
    ba[j] = 0.0f; bx[j] = 0.0f; by[j] = 0.0f; bz[j] = 0.0f; br[j] = 0.0f; bf[j] = 1.0f;
    bi[j] = 0u;
  }
  float T = 1.0f;
  uint32_t done = active ? 0u : 1u;  // a 0/1 vector register, as in render_tile
  for (uint32_t b = 0; b < len; b += kKBatchB) {
    if (__syncthreads_count(done == 0u) == 0) break;
    const uint32_t wb0 = b & ~(uint32_t)(kWinStep - 1), base = b & (kWin - 1);  // base: this batch's rows
    K.wlo = wb0 >= (uint32_t)kWinStep ? wb0 - kWinStep : 0u;
    if (t < kKBatchB) {
      // the rows of batch b - kWin have left the window (before the barrier above)
      if (b >= (uint32_t)kWin) kbuf_flush_row(base + t, K);
      uint32_t fl = 0u;
      if (b + t < len) {
        const uint32_t e = ids[rg.x + b + t];
        pew[base + t] = e;
        float* c = cw + 3 * (base + t);
        c[0] = rgb[3 * (size_t)e]; c[1] = rgb[3 * (size_t)e + 1]; c[2] = rgb[3 * (size_t)e + 2];
        fl = pair_setup<RS, true, GEN, CLIP>(record, rgb, e, (int)(e - (uint32_t)cam_idx * (uint32_t)n),
                                             F, cam, umax, vmax, dtmax, th, l2amin, wb, &pd[t * S]);
      }
      pf[t] = (unsigned short)fl;
    }
    __syncthreads();
    if (wave_any(done == 0u)) {
      const uint32_t lm = build_lists<RS, true>(pd, pf, wv, box, done == 0u, lists[wv]);
      const int cnt = (int)(lm & ~kMixed);
      const bool mixed = (lm & kMixed) != 0u;
      const unsigned char* mine = lists[wv].row[lane >> 4];
      for (int k = 0; k < cnt; k++) {
        if (!wave_any(done == 0u)) break;
        const uint32_t i = mine[k];  // (per row of lanes)
        const float4* P = pd + i * S;
        PairRegs<RS> r;
        load_pair<RS>(P, r);
        Eval ev;
        eval_test<RS>(r, P, u, v, dt, mixed, &ev);
        if (CLIP) clip_test<RS>(r, P, u, v, dt, dlen, clipv, &ev);
        const bool live = eval_hit<RS>(r, ev) && done == 0u;
        if (!wave_any(live)) continue;
        eval_alpha<RS, GEN>(r, th, &ev);
        float odg;
        if (!RS) {
          const float4 p5 = P[5];
          odg = fmaf(v, p5.z, fmaf(u, p5.y, p5.x));
        } else {
          odg = fmaf(v, r.p4.w, fmaf(u, r.p3.w, r.p5.w));
          odg = fmaf(dt, fmaf(v, r.p9.w, fmaf(u, r.p8.w, r.p7.w)), odg);
        }
        const float dist = -odg * dlen * ev.idd;
        const uint32_t pos = b + i;  // the hit's list position
        // the closest point p = d_g x (o_g x d_g) / |d_g|^2 and rho, as in render_bwd_kernel
        float3 dg, cr;
        pair_vectors<RS>(P, ev, u, v, &dg, &cr);
        float3 pv = cross3f_fma(dg, cr);
        pv = f3(pv.x * ev.idd, pv.y * ev.idd, pv.z * ev.idd);
        const float rho0 = ev.araw * __builtin_amdgcn_exp2f(-r.lsig);
        const float rho = ev.clamped ? -rho0 - 1e-30f : rho0;
        // degree n: d alpha / d omega^2 relative to the Gaussian's (as in render_bwd_kernel)
        const float fg = GEN ? __builtin_amdgcn_exp2f(fmaf(th.k_h - 1.0f, ev.lq, th.k_f)) : 1.0f;
        // a lane blends either the hit, if it lies at or before the buffer's
        // nearest, or that one, which the hit then displaces
        const bool ins = live && !(dist <= bd[0]);
        kbuf_blend_bwd(live, ins ? ba[0] : ev.a, ins ? bi[0] : pos, ins ? bx[0] : pv.x, ins ? by[0] : pv.y,
                       ins ? bz[0] : pv.z, ins ? br[0] : rho, ins ? bf[0] : fg, K, gC, gCd, gTT, T, Z, done);
        if (ins) {
#pragma unroll
          for (int j = 0; j < kKBufB - 1; j++) {
            const bool nx = bd[j + 1] < dist, here = j == 0 || bd[j] < dist;
            // sorted buffer and dist > bd[0]: the middle one of bd[j], dist, bd[j + 1]
            bd[j] = __builtin_amdgcn_fmed3f(bd[j], dist, bd[j + 1]);
            ba[j] = nx ? ba[j + 1] : (here ? ev.a : ba[j]);
            bi[j] = nx ? bi[j + 1] : (here ? pos : bi[j]);
            bx[j] = nx ? bx[j + 1] : (here ? pv.x : bx[j]);
            by[j] = nx ? by[j + 1] : (here ? pv.y : by[j]);
            bz[j] = nx ? bz[j + 1] : (here ? pv.z : bz[j]);
            br[j] = nx ? br[j + 1] : (here ? rho : br[j]);
            if (GEN) bf[j] = nx ? bf[j + 1] : (here ? fg : bf[j]);
          }
          const int L = kKBufB - 1;
          const bool last = bd[L] < dist;
          ba[L] = last ? ev.a : ba[L];
          bi[L] = last ? pos : bi[L];
          bx[L] = last ? pv.x : bx[L];
          by[L] = last ? pv.y : by[L];
          bz[L] = last ? pv.z : bz[L];
          br[L] = last ? rho : br[L];
          if (GEN) bf[L] = last ? fg : bf[L];
          bd[L] = last ? dist : bd[L];
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kKBufB; j++)
    kbuf_blend_bwd(true, ba[j], bi[j], bx[j], by[j], bz[j], br[j], bf[j], K, gC, gCd, gTT, T, Z, done);
  __syncthreads();
  for (int r = t; r < kWin; r += kKThreadsB) kbuf_flush_row(r, K);
}

// K7a: camera-independent part of the per-particle chain (FP64: the
// quaternion gradient is a difference of terms of the size of dL/dR).
__global__ void particle_grad_kernel(int n, const float* __restrict__ scales,
                                     const float* __restrict__ quats, const double* __restrict__ acc,
                                     float* __restrict__ g_means, float* __restrict__ g_scales,
                                     float* __restrict__ g_quats, float* __restrict__ g_opac) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double* a = acc + (long long)i * kAcc;
  const double G[9] = {a[0], a[1], a[2], a[1], a[3], a[4], a[2], a[4], a[5]};
  const double h[3] = {a[6], a[7], a[8]};
  const double s[3] = {scales[3 * i], scales[3 * i + 1], scales[3 * i + 2]};
  const float4 qf = reinterpret_cast<const float4*>(quats)[i];
  // R(q / |q|), q = (w, x, y, z)
  const double qn = sqrt((double)qf.x * qf.x + (double)qf.y * qf.y + (double)qf.z * qf.z +
                         (double)qf.w * qf.w);
  const double iq = 1.0 / qn;
  const double w = qf.x * iq, x = qf.y * iq, y = qf.z * iq, z = qf.w * iq;
  const double R[9] = {1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)};
  // dL/ds_k = -G_kk / s_k
  g_scales[3 * i] = (float)(-G[0] / s[0]);
  g_scales[3 * i + 1] = (float)(-G[4] / s[1]);
  g_scales[3 * i + 2] = (float)(-G[8] / s[2]);
  // dL/dmu = -R S^-1 h
  const double hs[3] = {h[0] / s[0], h[1] / s[1], h[2] / s[2]};
  for (int r = 0; r < 3; r++)
    g_means[3 * i + r] = (float)(-(R[3 * r] * hs[0] + R[3 * r + 1] * hs[1] + R[3 * r + 2] * hs[2]));
  // dL/dR = R S G S^-1
  double X[9];  // S G S^-1
  for (int l = 0; l < 3; l++)
    for (int k = 0; k < 3; k++) X[3 * l + k] = s[l] * G[3 * l + k] / s[k];
  double gR[9];
  for (int j = 0; j < 3; j++)
    for (int k = 0; k < 3; k++)
      gR[3 * j + k] = R[3 * j] * X[k] + R[3 * j + 1] * X[3 + k] + R[3 * j + 2] * X[6 + k];
  // through R(q/|q|):  R entries are quadratic in (w, x, y, z)
  const double gw = 2 * (x * (gR[7] - gR[5]) + y * (gR[2] - gR[6]) + z * (gR[3] - gR[1]));
  const double gx = 2 * (w * (gR[7] - gR[5]) + y * (gR[1] + gR[3]) + z * (gR[2] + gR[6]) -
                         2 * x * (gR[4] + gR[8]));
  const double gy = 2 * (w * (gR[2] - gR[6]) + x * (gR[1] + gR[3]) + z * (gR[5] + gR[7]) -
                         2 * y * (gR[0] + gR[8]));
  const double gz = 2 * (w * (gR[3] - gR[1]) + x * (gR[2] + gR[6]) + y * (gR[5] + gR[7]) -
                         2 * z * (gR[0] + gR[4]));
  const double pdot = w * gw + x * gx + y * gy + z * gz;
  reinterpret_cast<float4*>(g_quats)[i] =
      make_float4((float)((gw - w * pdot) * iq), (float)((gx - x * pdot) * iq),
                  (float)((gy - y * pdot) * iq), (float)((gz - z * pdot) * iq));
  g_opac[i] = (float)a[9];
}

// K7b: SH colour of one camera -> dL/dbeta and dL/dmu through the view
// direction.  One thread per particle, 256 per block.  The block's
// coefficients (3K floats per particle, one contiguous slab) come in and its
// gradients go out as contiguous runs through LDS, at a padded stride so each
// thread's own row hits distinct banks; every global access is coalesced and
// all of a thread's loads are issued before any is used.  The first camera
// writes g_sh (zeros for particles without colour gradient), later cameras
// add to it.
constexpr int kShThreads = 256;

template <int DEG>
__global__ void __launch_bounds__(kShThreads) sh_grad_kernel(
    int n, int cam_idx, int first, DevCam cam, Thresholds th, const float* __restrict__ means,
    const float* __restrict__ sh, const float* __restrict__ rgb, const double* __restrict__ acc_rgb,
    float* __restrict__ g_means, float* __restrict__ g_sh) {
  constexpr int K = (DEG + 1) * (DEG + 1), C = 3 * K, LD = C + 1;
  constexpr int kPer = C;  // slab floats per thread (C * 256 / 256)
  __shared__ float lb[kShThreads * LD];
  const int t = threadIdx.x;
  const long long i0 = (long long)blockIdx.x * kShThreads;
  const int cnt = (int)min((long long)kShThreads, (long long)n - i0);
  const long long i = i0 + t;
  float gr[3] = {0.f, 0.f, 0.f};
  bool live[3] = {false, false, false};
  if (t < cnt) {
    const long long e = (long long)cam_idx * n + i;
    for (int c = 0; c < 3; c++) {
      gr[c] = (float)acc_rgb[3 * e + c];
      live[c] = gr[c] != 0.0f && rgb[3 * e + c] > 0.0f;  // max(0, .) clamps the rest
    }
  }
  const bool any = live[0] || live[1] || live[2];
  const bool block_any = __syncthreads_or(any);
  if (!block_any && !first) return;  // nothing to add for these particles
  const float* src = sh + i0 * C;
  float* dst = g_sh + i0 * C;
  const int m = cnt * C;  // slab length
  if (block_any) {
    float v[kPer];
#pragma unroll
    for (int q = 0; q < kPer; q++) {
      const int j = t + q * kShThreads;
      v[q] = j < m ? src[j] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < kPer; q++) {
      const int j = t + q * kShThreads;
      lb[(j / C) * LD + j % C] = v[q];
    }
  }
  __syncthreads();
  float gs[C];
#pragma unroll
  for (int k = 0; k < C; k++) gs[k] = 0.0f;
  if (any) {
    float3 mu = f3(means[3 * i], means[3 * i + 1], means[3 * i + 2]);
    float t0 = 0.0f;
    if (cam.shutter == GUT_ROLLING_TOP_TO_BOTTOM) {  // exposure time of the mean, as in K1
      float2 vv;
      bool ok;
      t0 = solve_project(cam, cam0_coords(cam, mu), th, &vv, &ok);
    }
    float3 ctr = centre_at(cam, t0);
    float3 dv = f3(mu.x - ctr.x, mu.y - ctr.y, mu.z - ctr.z);
    float dist = sqrtf(dot3f(dv, dv)), id = 1.0f / dist;
    float3 d = f3(dv.x * id, dv.y * id, dv.z * id);
    float Y[K];
    float3 dY[K];
    sh_basis<DEG>(d.x, d.y, d.z, Y);
    sh_basis_grad<DEG>(d.x, d.y, d.z, dY);
    const float* b = lb + t * LD;
    float3 gd = f3(0.f, 0.f, 0.f);
#pragma unroll
    for (int c = 0; c < 3; c++) {
      const float g = live[c] ? gr[c] : 0.0f;
#pragma unroll
      for (int k = 0; k < K; k++) {
        gs[3 * k + c] = g * Y[k];
        const float bb = g * b[3 * k + c];
        gd = f3(gd.x + bb * dY[k].x, gd.y + bb * dY[k].y, gd.z + bb * dY[k].z);
      }
    }
    float pdd = dot3f(gd, d);
    g_means[3 * i] += (gd.x - d.x * pdd) * id;
    g_means[3 * i + 1] += (gd.y - d.y * pdd) * id;
    g_means[3 * i + 2] += (gd.z - d.z * pdd) * id;
  }
  __syncthreads();  // the coefficients are read; the same LDS takes the gradients
#pragma unroll
  for (int k = 0; k < C; k++) lb[t * LD + k] = gs[k];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; q++) {
    const int j = t + q * kShThreads;
    if (j >= m) continue;
    const float g = lb[(j / C) * LD + j % C];
    dst[j] = first ? g : dst[j] + g;
  }
}

__global__ void zero_f64_kernel(double* __restrict__ p, long long m) {
  long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < m) p[j] = 0.0;
}

}  // namespace gut

using namespace gut;

extern "C" size_t gut_render_bwd_workspace_bytes(int64_t n, int32_t n_cams) {
  if (n < 0 || n_cams <= 0) return 0;
  size_t a = ((size_t)n * kAcc * 8 + 255) & ~size_t(255);
  return a + (size_t)n * n_cams * 3 * 8 + 256;
}

// Whether the tile-order backward of a camera of this many tiles takes pairs
// (128 threads, two pixels a thread) or lists.  Lists reach fewer pixels in
// vain and spread a tile's walk over twice the waves; pairs sum twice the pixels
// in a step, which wins where few small particles lie on a tile: each then
// covers its quadrants, or the launch's fixed work a tile counts most.  us a
// backward, lists (pairs); "large" are particles of several quadrants:
//   1200 tiles   2k large 132 (157), 100k 113 (245)
//   2560         2k large 220 (218), rolling 121 (145)
//   3600         2k large 283 (273), rolling 161 (148); 20k large 338 (314),
//                rolling 181 (196); 100k 157 (164), rolling 163 (364)
//   7500         20k large 608 (527); 100k 257 (250), rolling 246 (293)
//   8160         20k large 647 (577), rolling 342 (308); 100k 286 (262), rolling
//                269 (270); 1M 894 (937), fisheye 819 (941), rolling 881 (1014)
//   14400        100k 442 (373); 1M 1348 (1319), fisheye 1131 (1232)
//   32400        200k large 2397 (2032); 1M 2573 (2342), fisheye 1979 (1982)
// So lists below 3072 tiles and from tiles / 650 particles a tile on.
static bool bwd_by_pairs(int64_t tiles, int64_t n) { return tiles >= 3072 && 650 * n < tiles * tiles; }

// The whole backward with its FP64 accumulators in ws (ws_bytes available):
// argument checks, then every launch on `stream`.
static gut_status render_bwd_run(const gut_scene* scene, const gut_projected* proj,
                                 const uint32_t* tile_ranges, const uint32_t* sorted_ids,
                                 const gut_camera* cams, int32_t n_cams, const gut_params* p,
                                 const float* clip_depth, const float* rgb, const float* T_final,
                                 const uint32_t* n_contrib, const float* d_rgb, const float* d_T,
                                 float* g_means, float* g_scales, float* g_quats,
                                 float* g_opacities, float* g_sh, void* ws, size_t ws_bytes,
                                 void* stream) {
  gut_status st = check_params(p);
  if (st != GUT_OK) return st;
  if ((st = check_scene(scene, true)) != GUT_OK) return st;
  if (!proj || !proj->record || !proj->rgb || !tile_ranges || !rgb || !T_final || !n_contrib ||
      !d_rgb || !g_means || !g_scales || !g_quats || !g_opacities || !g_sh) {
    set_error("gut_render_bwd: a required pointer is NULL");
    return GUT_E_INVALID;
  }
  if (((uintptr_t)proj->record & 15) || ((uintptr_t)scene->quats & 15) ||
      ((uintptr_t)g_quats & 15) || ((uintptr_t)tile_ranges & 7)) {
    set_error("record, quats, g_quats must be 16-byte and tile_ranges 8-byte aligned");
    return GUT_E_INVALID;
  }
  const int64_t n = scene->n;
  if (n * (int64_t)n_cams >= (int64_t(1) << 31)) {
    set_error("n * n_cams must be below 2^31");
    return GUT_E_INVALID;
  }
  size_t need = gut_render_bwd_workspace_bytes(n, n_cams);
  if (!ws || ws_bytes < need || ((uintptr_t)ws & 255)) {
    set_error("workspace must be 256-byte aligned and hold %zu bytes", need);
    return GUT_E_INVALID;
  }
  DevCam dc[kMaxCams];
  int64_t T = 0;
  if ((st = prepare_cams(cams, n_cams, *p, dc, &T, nullptr)) != GUT_OK) return st;
  if (n == 0) return GUT_OK;
  const uint32_t* order = tile_ranges + 2 * T;
  hipStream_t s = (hipStream_t)stream;
  double* acc = (double*)ws;
  double* acc_rgb = (double*)((char*)ws + (((size_t)n * kAcc * 8 + 255) & ~size_t(255)));
  long long m1 = n * kAcc, m2 = n * n_cams * 3;
  zero_f64_kernel<<<(unsigned)((m1 + 255) / 256), 256, 0, s>>>(acc, m1);
  GUT_LAUNCH_CHECK();
  zero_f64_kernel<<<(unsigned)((m2 + 255) / 256), 256, 0, s>>>(acc_rgb, m2);
  GUT_LAUNCH_CHECK();
  Thresholds th = make_thresholds(*p);
  for (int c = 0; c < n_cams && p->kbuffer > 0; c++) {  // "Ours (sorted)"
    dim3 grid(dc[c].tiles_x * dc[c].tiles_y), block(kKThreadsB);
#define GUT_KBW(RS, GEN, CLIP)                                                                      \
  render_kbuffer_bwd_kernel<RS, GEN, CLIP><<<grid, block, 0, s>>>(                                   \
      dc[c], th, (int)n, c, p->kbuffer, (const uint2*)tile_ranges, order, sorted_ids,                 \
      (const float4*)proj->record, proj->rgb, clip_depth, rgb, T_final, d_rgb, d_T, acc, acc_rgb)
#define GUT_KBW1(RS, GEN) \
  do { if (clip_depth) GUT_KBW(RS, GEN, true); else GUT_KBW(RS, GEN, false); } while (0)
    const bool rs = dc[c].shutter == GUT_ROLLING_TOP_TO_BOTTOM, gen = th.kdeg != 2;
    if (rs) { if (gen) GUT_KBW1(true, true); else GUT_KBW1(true, false); }
    else { if (gen) GUT_KBW1(false, true); else GUT_KBW1(false, false); }
#undef GUT_KBW1
#undef GUT_KBW
    GUT_LAUNCH_CHECK();
  }
  for (int c = 0; c < n_cams && p->kbuffer == 0; c++) {
    dim3 grid(dc[c].tiles_x * dc[c].tiles_y);
    const bool pairs = bwd_by_pairs(grid.x, n);
#define GUT_RBWK(K, NT, RS, GEN, CLIP)                                                               \
  K<RS, GEN, CLIP><<<grid, NT, 0, s>>>(                                                              \
      dc[c], th, (int)n, c, (const uint2*)tile_ranges, order, sorted_ids,                         \
      (const float4*)proj->record, clip_depth, proj->rgb, rgb, T_final, n_contrib, d_rgb, d_T, acc, acc_rgb)
#define GUT_RBW(RS, GEN, CLIP)                                                            \
  do {                                                                                    \
    if (pairs) GUT_RBWK(render_bwd_pairs_kernel, kBpThreads, RS, GEN, CLIP);              \
    else GUT_RBWK(render_bwd_kernel, kBwThreads, RS, GEN, CLIP);                          \
  } while (0)
#define GUT_RBW1(RS, GEN) \
  if (clip_depth) GUT_RBW(RS, GEN, true); else GUT_RBW(RS, GEN, false)
    const bool gen = th.kdeg != 2;
    if (dc[c].shutter == GUT_ROLLING_TOP_TO_BOTTOM) { if (gen) { GUT_RBW1(true, true); } else { GUT_RBW1(true, false); } }
    else { if (gen) { GUT_RBW1(false, true); } else { GUT_RBW1(false, false); } }
#undef GUT_RBW1
#undef GUT_RBW
#undef GUT_RBWK
    GUT_LAUNCH_CHECK();
  }
  dim3 g1((unsigned)((n + 255) / 256)), b1(256);
  particle_grad_kernel<<<g1, b1, 0, s>>>((int)n, scene->scales, scene->quats, acc, g_means,
                                         g_scales, g_quats, g_opacities);
  GUT_LAUNCH_CHECK();
  const dim3 gs_grid((unsigned)((n + kShThreads - 1) / kShThreads));
  for (int c = 0; c < n_cams; c++) {
#define GUT_SHG(D)                                                                          \
  sh_grad_kernel<D><<<gs_grid, kShThreads, 0, s>>>((int)n, c, c == 0, dc[c], th, scene->means, \
                                                   scene->sh, proj->rgb, acc_rgb, g_means, g_sh)
    switch (scene->sh_degree) {
      case 0: GUT_SHG(0); break;
      case 1: GUT_SHG(1); break;
      case 2: GUT_SHG(2); break;
      default: GUT_SHG(3); break;
    }
#undef GUT_SHG
    GUT_LAUNCH_CHECK();
  }
  return GUT_OK;
}

extern "C" gut_status gut_render_bwd(const gut_scene* scene, const gut_projected* proj,
                                     const uint32_t* tile_ranges, const uint32_t* sorted_ids,
                                     const gut_camera* cams, int32_t n_cams, const gut_params* p,
                                     const float* clip_depth, const float* rgb, const float* T_final,
                                     const uint32_t* n_contrib, const float* d_rgb,
                                     const float* d_T, float* g_means, float* g_scales,
                                     float* g_quats, float* g_opacities, float* g_sh, void* ws,
                                     size_t ws_bytes, void* stream) {
  return render_bwd_run(scene, proj, tile_ranges, sorted_ids, cams, n_cams, p, clip_depth, rgb,
                        T_final, n_contrib, d_rgb, d_T, g_means, g_scales, g_quats, g_opacities,
                        g_sh, ws, ws_bytes, stream);
}

// ---- the backward without a caller workspace --------------------------------
// For callers that cannot allocate (graph capture, serving loops, harnesses
// that forbid it): the FP64 accumulators live in one static device array per
// GPU, held from the library's load until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is only a stand-in);
// its device address is looked up once per device, with that device current,
// and kept.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};

gut_status scratch_address(void** out) {
  int dev = 0;
  GUT_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxScratchDevices) {
    set_error("gut_render_bwd_noalloc: device %d is beyond the %d supported", dev,
              kMaxScratchDevices);
    return GUT_E_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    GUT_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr || ((uintptr_t)ptr & 255)) {
      set_error("gut_render_bwd_noalloc: scratch address %p is not 256-byte aligned", ptr);
      return GUT_E_HIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return GUT_OK;
}
}  // namespace

extern "C" gut_status gut_render_bwd_noalloc(const gut_scene* scene, const gut_projected* proj,
                                             const uint32_t* tile_ranges, const uint32_t* sorted_ids,
                                             const gut_camera* cams, int32_t n_cams,
                                             const gut_params* p, const float* clip_depth,
                                             const float* rgb, const float* T_final,
                                             const uint32_t* n_contrib, const float* d_rgb,
                                             const float* d_T, float* g_means, float* g_scales,
                                             float* g_quats, float* g_opacities, float* g_sh,
                                             void* stream) {
  if (!scene || scene->n < 0 || n_cams <= 0) {
    set_error("gut_render_bwd_noalloc: NULL scene, n < 0 or n_cams <= 0");
    return GUT_E_INVALID;
  }
  const size_t need = gut_render_bwd_workspace_bytes(scene->n, n_cams);
  if (need > kNoAllocScratchBytes) {
    set_error("gut_render_bwd_noalloc: n = %lld particles over %d camera(s) need %zu bytes of "
              "scratch; the static scratch holds %zu (use gut_render_bwd with a workspace)",
              (long long)scene->n, (int)n_cams, need, kNoAllocScratchBytes);
    return GUT_E_INVALID;
  }
  void* ws = nullptr;
  gut_status st = scratch_address(&ws);
  if (st != GUT_OK) return st;
  return render_bwd_run(scene, proj, tile_ranges, sorted_ids, cams, n_cams, p, clip_depth, rgb,
                        T_final, n_contrib, d_rgb, d_T, g_means, g_scales, g_quats, g_opacities,
                        g_sh, ws, kNoAllocScratchBytes, stream);
}
