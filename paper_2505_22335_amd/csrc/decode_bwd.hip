// Decoder backward on the matrix cores (VJP of UP-SLAM Eq. 8 and Eq. 9), all
// views in one launch. One workgroup of eight waves takes (16-anchor tile,
// view) items in turn, a tile's views one after another: waves 0..3 each own
// one of the opacity, colour, scale and rotation heads, waves 4..7 share the
// feature head's output rows. Per item and head, with X the item's inputs (one
// row per anchor):
//   Z = X W1^T + b1, H = act(Z)                 (ReLU; SoftPlus for features)
//   Y = H W2^T + b2, dY = dL/d(decoded) * act'(Y)
//   dW2 += dY^T H, db2 += sum_a dY, dH = dY W2, dZ = dH * act'(Z)
//   dW1 += dZ^T X, db1 += sum_a dZ, dX = dZ W1
// all on FP32 16x16x4 MFMAs. The heads' dX are summed per anchor in a fixed
// order inside the workgroup, which then forms the anchor gradients (feature
// part; view direction and distance through delta = (x - c)/|x - c|) and its
// share of the camera-centre gradient. Each workgroup keeps one partial of
// every parameter gradient, reduced afterwards in a fixed order
// (deterministic, no atomics). An item's products over its anchors are summed
// on their own and added to the running sums as one number, and the running
// sums go into the partial after every kChainViews views' worth of items:
// rounded after every four anchors and over all views, the gradients of two
// views of 33k anchors were 2.8e-7 of their norm away from FP64, of sixteen
// views of 500 3.0e-7; so 1.4e-7 and 1.3e-7, for 5 % of the time.
//
// The workgroup meets at one barrier per item. What crosses waves is taken up
// one item later: the feature waves' dH partials (then the feature head's dX
// and dW1), the rotation head's dZ (its dW1 is wave 4's), and, after the
// barrier, the sum of the heads' dX. Every feature wave forms the feature
// head's hidden layer itself. So the two waves of a SIMD drift apart and one's
// matrix products run under the other's activations and LDS traffic; each
// SIMD's pair has about 204 products (32 cycles each) per item at k = 10, 6.5k
// of the roughly 11k cycles an item takes (16k with three barriers per item
// and the head's activation chosen per element). One launch per view, each
// with its own prologue and parameter partials, took 116 us a view for 50k
// anchors (eight views 931 us, now 565); one view of 100k anchors 180 us, now
// 156; of 20k 50 us, now 46; of 20k with k = 16 and its reduction 71 us, now 60.
//
// Operand layouts. v_mfma_f32_16x16x4f32 (wave64): lane l = 16 g + f supplies
// A[f][g] and B[g][f] and receives D[4 g + r][f], r = 0..3. A 16x16 block
// held by rows in that way (lane (f, g) holds M[4 g + r][f]) is directly a B
// operand with K = its rows, and an A operand with K = its rows and M = its
// columns, when step r of lane group g takes K index 4 g + r (a contraction
// may visit K in any order that both operands share). Chained this way, H and
// dH stay in registers as (units x anchors) blocks and Y, dY as (anchors x
// rows) blocks; only H, dY and dZ pass once each through per-wave LDS rows to
// be transposed. Both layouts of the second-layer weights (B of Y, A of dH^T)
// sit in registers for the whole kernel; the first-layer weights (A of Z^T
// and of dX^T) are read from LDS, as are the tile's inputs and upstream
// gradients, which are loaded a tile ahead as coalesced runs.
#include <math.h>

#include <type_traits>

#include "decode_shared.h"

namespace asgs {

namespace {

typedef float f4v __attribute__((ext_vector_type(4)));

constexpr int kBW = 8;         // waves per workgroup
constexpr int kBT = 64 * kBW;  // threads per workgroup
constexpr int kMaxWG = 256;    // one workgroup per compute unit
constexpr int kChainViews = 4; // views' worth of items summed before they go into the partial
constexpr int kW1L = 36;       // LDS row of a first-layer weight row: 35 inputs + the distance column
constexpr int kW2L = 36;       // LDS row of a second-layer weight row in the prologue (32 units + pad)
constexpr int kXL = 52;        // LDS row of an anchor's inputs: 35 + distance column, |x - c| at 36
constexpr int kHB = 36;        // per-wave transpose rows of H, dZ (32 units + pad) and two row tiles of dY
constexpr int kDXL = 36;       // dX row of an anchor in a head's slot

constexpr int kPlanes = 27;    // (head, component) planes of the upstream gradients: 1 + 3 + 3 + 4 + 16

// LDS carve (floats); kR: second-layer row tiles per wave
template <int kR>
struct Lds {
  static constexpr int kMaxK = kR == 3 ? 12 : ASGS_MAX_K;                 // largest k of this instantiation
  static constexpr int kW1 = 0;                                           // [5 heads][32][kW1L]
  static constexpr int kX = kW1 + kHeads * kHid * kW1L;                   // three items' inputs
  static constexpr int kTW = kX + 3 * 16 * kXL;                           // temporal weights [2][5 heads][32]
  static constexpr int kDC = kTW + 2 * kHeads * kHid;                     // camera-centre sums [views][3]
  static constexpr int kHBo = kDC + 3 * ASGS_MAX_VIEWS;                   // per wave: transpose rows (H, dY, dZ)
  static constexpr int kHR = kHBo + kBW * 16 * kHB;                       // the rotation head's dZ, two items
  static constexpr int kDH = kHR + 2 * 16 * kHB;                          // feature dH partials, two items
  static constexpr int kDX = kDH + 2 * 4 * 64 * 8;                        // dX of heads 0..3, three items
  static constexpr int kDXF = kDX + 3 * 4 * 16 * kDXL;                    // dX of the feature head, two items
  static constexpr int kG = kDXF + 2 * 16 * kDXL;
  static constexpr int kGB = kPlanes * (16 * kMaxK + 1);  // upstream gradients, two items: each plane's run of 16 k values + pad
  static constexpr int kFloats = kG + 2 * kGB;
  // the second-layer weights (at most 27 k rows of kW2L), b2 and b1 are copied
  // once into the region from kHBo on
  static_assert(kFloats - kHBo >= 27 * kMaxK * (kW2L + 1) + 3 + kHeads * kHid, "weight copy does not fit");
  static_assert(kFloats * 4 <= 160 * 1024, "LDS");
};

ASGS_DEV f4v mfma(float a, float b, f4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

ASGS_DEV void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int kR>
__global__ void __launch_bounds__(kBT, 1) k_dec_bwd(DecodeConst dc, HeadTable ht, DecodeViews dv,
                                                    const float* __restrict__ xyz, const float* __restrict__ feat,
                                                    const float* __restrict__ params, PlaneTable pt,
                                                    DecWork w, float* d_xyz, float* d_feat, int want_params) {
  using C = Lds<kR>;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int fl = lane & 15, fg = lane >> 4;
  float* const W1L = smem + C::kW1;
  float (*const XB)[16][kXL] = reinterpret_cast<float (*)[16][kXL]>(smem + C::kX);
  float* const TW = smem + C::kTW;
  float* const DC = smem + C::kDC;
  float (*const HBw)[kHB] = reinterpret_cast<float (*)[kHB]>(smem + C::kHBo + wv * 16 * kHB);
  float (*const HR)[16][kHB] = reinterpret_cast<float (*)[16][kHB]>(smem + C::kHR);
  float* const DH = smem + C::kDH;
  float (*const DX)[4][16][kDXL] = reinterpret_cast<float (*)[4][16][kDXL]>(smem + C::kDX);
  float (*const DXF)[16][kDXL] = reinterpret_cast<float (*)[16][kDXL]>(smem + C::kDXF);
  float* const GB = smem + C::kG;
  const int A = (int)dc.A;
  const int k = dc.k;
  const int n = A * k;
  const int nx = ht.nx;
  const int V = dc.n_views;
  const bool has_feat = ht.m[4] > 0;
  // ---- this wave's head, output rows and duties ----
  const int hd = wv < 4 ? wv : 4;
  const int q = wv - 4;  // index among the feature waves
  const bool active = wv < 4 || has_feat;
  const int m = ht.m[hd];
  const int rows = k * m;
  const int T = (rows + 15) / 16;
  int t0 = 0, nt = T;
  if (wv >= 4) {
    const int base = T / 4, extra = T - 4 * base;
    nt = base + (q < extra ? 1 : 0);
    t0 = q * base + (q < extra ? q : extra);
  }
  // dX: waves 0..3 and feature wave 2. dW1, db1: waves 0..2 of their heads,
  // feature wave 0 of the rotation head (its wave has the most rows) and
  // feature wave 3 of the feature head
  const int hw1 = wv < 3 ? wv : wv == 4 ? 3 : (wv == 7 && has_feat) ? 4 : -1;
  const int w2o = (int)ht.off[hd] + kHid * kIn + kHid;  // the head's W2 [rows][32], then b2 [rows]
  // the tile's upstream gradients are staged per (head, component) plane as
  // runs of 16 k values (stride run + 1, odd, against bank conflicts)
  const int run = 16 * k, gstride = run + 1;
  // ---- per-item inputs: features, positions and upstream gradients, fetched an
  // item ahead into registers and staged through LDS ----
  // (loads into registers are unconditional, from clamped indices, and masked
  // when staged: a load under a branch would be waited for at the branch's end)
  float xv = 0.f, pv[3] = {0.f, 0.f, 0.f};
  auto fetch_x = [&](int tile) {
    const int a0 = tile * 16, a = t >> 5, c = t & 31;
    const int ax = a0 + a < A ? a0 + a : 0, ap = a0 + (t & 15) < A ? a0 + (t & 15) : 0;
    xv = feat[(int64_t)ax * 32 + c];
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) pv[cc] = xyz[(int64_t)cc * A + ap];
  };
  auto put_x = [&](int buf, int tile, int view) {
    const int a0 = tile * 16;
    XB[buf][t >> 5][t & 31] = a0 + (t >> 5) < A ? xv : 0.f;
    if (wv == 0) {
      // lane 16 c + a: component c of anchor a's direction; lanes 48 + a: its distance
      const bool ok = a0 + fl < A;
      float D[3];
      for (int c = 0; c < 3; ++c) D[c] = pv[c] - dv.c[view][c];
      const float dist = ok ? sqrtf(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]) : 1.f;
      const float dc_ = fg == 0 ? D[0] : fg == 1 ? D[1] : D[2];
      const float del = ok ? dc_ / dist : 0.f;
      if (fg < 3) {
        XB[buf][fl][32 + fg] = del;
      } else {
        XB[buf][fl][35] = nx > 0 && ok ? dist : 0.f;  // distance input (weight column 35)
        XB[buf][fl][36] = dist;                       // |x - c| for the anchor gradients
      }
    }
  };
  // wave w loads planes w, w + 8, w + 16, w + 24, each as kR coalesced chunks of
  // 64 values (16 k <= 64 kR) at 32-bit offsets from the plane; values past the
  // last anchor repeat the plane's last one and are masked where they are used
  const int nplanes = has_feat ? kPlanes : 11;
  float gpre[4][kR];
  auto fetch_g = [&](int tile, int view) {
    uint32_t off[kR];
#pragma unroll
    for (int c = 0; c < kR; ++c) off[c] = 4u * (uint32_t)min(tile * run + lane + 64 * c, n - 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int p = wv + 8 * i < nplanes ? wv + 8 * i : 0;
      const char* src = reinterpret_cast<const char*>(pt.base[p] + view * pt.stride[p]);
#pragma unroll
      for (int c = 0; c < kR; ++c) gpre[i][c] = *reinterpret_cast<const float*>(src + off[c]);
    }
  };
  auto put_g = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (wv + 8 * i >= nplanes) break;
      float* dst = GB + buf * C::kGB + (wv + 8 * i) * gstride + lane;
#pragma unroll
      for (int c = 0; c < kR; ++c)
        if (lane + 64 * c < run) dst[64 * c] = gpre[i][c];
    }
  };
  const int ngrid = (A + 15) / 16;
  if ((int)blockIdx.x < ngrid) {
    fetch_x(blockIdx.x);
    fetch_g(blockIdx.x, 0);
  }
  // ---- the weights into LDS (coalesced): the first-layer rows of every head
  // (kept for the whole kernel); the second-layer rows (36 floats: b128 reads
  // of four units and b32 reads across rows without bank conflicts), b2 and
  // b1, in the region past the input tiles, which is free until the first item
  // is staged ----
  float* const W2L = smem + C::kHBo;                         // [all rows][kW2L]
  const int nrows = ht.nrows;
  float* const B2L = W2L + nrows * kW2L;                    // [all rows]
  float* const B1L = B2L + ((nrows + 3) & ~3);             // [5 heads][32] (16-byte aligned)
  {
    // head by head, each a contiguous block of the packed parameters: every
    // load of the thread is issued before its first store
    constexpr int kK = C::kMaxK;
    constexpr int kMs[kHeads] = {1, 3, 3, 4, 16};
    constexpr int kE1 = (kHid * kIn + kBT - 1) / kBT;
    constexpr int kE2m = (16 * kK * kHid + kBT - 1) / kBT;
    const int nh = has_feat ? kHeads : 4;
    float v1[kHeads][kE1], v2[kHeads][kE2m], vd[kHeads], vb1[kHeads], vb2[kHeads], vt0[kHeads], vt1[kHeads];
#pragma unroll
    for (int h = 0; h < kHeads; ++h) {
      if (h >= nh) break;
      const int o1 = (int)ht.off[h], rw = k * ht.m[h], w2 = o1 + kHid * kIn + kHid;
      const int ox = (int)ht.xoff[h];
#pragma unroll
      for (int q = 0; q < kE1; ++q) {
        const int e = t + q * kBT;
        v1[h][q] = params[o1 + (e < kHid * kIn ? e : 0)];
      }
      const int ne2 = (kMs[h] * kK * kHid + kBT - 1) / kBT;  // a constant once unrolled
#pragma unroll
      for (int q = 0; q < kE2m; ++q) {
        if (q >= ne2) break;
        const int e = t + q * kBT;
        v2[h][q] = params[w2 + (e < rw * kHid ? e : 0)];
      }
      vd[h] = nx > 0 ? params[ox + (t & 31) * nx] : 0.f;
      vb1[h] = params[o1 + kHid * kIn + (t & 31)];
      vt0[h] = nx == 3 ? params[ox + (t & 31) * 3 + 1] : 0.f;
      vt1[h] = nx == 3 ? params[ox + (t & 31) * 3 + 2] : 0.f;
      vb2[h] = params[w2 + rw * kHid + (t < rw ? t : 0)];
    }
#pragma unroll
    for (int h = 0; h < kHeads; ++h) {
      if (h >= nh) break;
      const int rw = k * ht.m[h], r0 = ht.row0[h];
#pragma unroll
      for (int q = 0; q < kE1; ++q) {
        const int e = t + q * kBT;
        const int u = e / kIn, i = e - u * kIn;
        if (e < kHid * kIn) W1L[(h * kHid + u) * kW1L + i] = v1[h][q];
      }
      const int ne2 = (kMs[h] * kK * kHid + kBT - 1) / kBT;
#pragma unroll
      for (int q = 0; q < kE2m; ++q) {
        if (q >= ne2) break;
        const int e = t + q * kBT;
        if (e < rw * kHid) W2L[(r0 + (e >> 5)) * kW2L + (e & 31)] = v2[h][q];
      }
      if (t < kHid) {
        W1L[(h * kHid + t) * kW1L + kIn] = vd[h];  // the distance weight (zero without that input)
        B1L[h * kHid + t] = vb1[h];
        TW[h * kHid + t] = vt0[h];
        TW[(kHeads + h) * kHid + t] = vt1[h];
      }
      if (t < rw) B2L[r0 + t] = vb2[h];
    }
    // input columns past 36 only meet discarded outputs of dW1; keep them finite
    for (int e = t; e < 3 * 16 * (kXL - 37); e += kBT) {
      const int row = e / (kXL - 37);
      XB[row >> 4][row & 15][37 + e - row * (kXL - 37)] = 0.f;
    }
    if (t < 3 * ASGS_MAX_VIEWS) DC[t] = 0.f;
  }
  __syncthreads();
  // ---- second-layer weights and biases in registers ----
  float b1r[2][4];
  float w2y[kR][2][4], w2h[kR][2][4], b2r[kR];
  // the lane's output row of row tile i reads plane offset goff[i] + a k
  const int pb0 = hd == 0 ? 0 : hd == 1 ? 1 : hd == 2 ? 4 : hd == 3 ? 7 : 11;  // first plane of the head
  const int hr0 = ht.row0[hd];  // the head's first row among all rows
  const int minv = (65536 + m - 1) / (m > 0 ? m : 1);  // o / m = (o * minv) >> 16, exact for o <= 256
  int goff[kR];
  bool rok[kR];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const f4v v = *reinterpret_cast<const f4v*>(&B1L[hd * kHid + 16 * b + 4 * fg]);
#pragma unroll
    for (int r = 0; r < 4; ++r) b1r[b][r] = active ? v[r] : 0.f;
  }
#pragma unroll
  for (int i = 0; i < kR; ++i) {
    const int o = 16 * (t0 + i) + fl;
    const bool ok = active && i < nt && o < rows;
    rok[i] = ok;
    const int oc = ok ? o : 0;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const f4v v = *reinterpret_cast<const f4v*>(&W2L[(hr0 + oc) * kW2L + 16 * b + 4 * fg]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int oh = 16 * (t0 + i) + 4 * fg + r;
        const bool okh = active && i < nt && oh < rows;
        w2y[i][b][r] = ok ? v[r] : 0.f;
        const float wh = W2L[(hr0 + (okh ? oh : 0)) * kW2L + 16 * b + fl];
        w2h[i][b][r] = okh ? wh : 0.f;
      }
    }
    b2r[i] = ok ? B2L[hr0 + oc] : 0.f;
    const int gi = (oc * minv) >> 16, gc = oc - gi * m;
    goff[i] = (pb0 + gc) * gstride + gi;
  }
  __syncthreads();  // the second-layer copy is no longer read
  if ((int)blockIdx.x < ngrid) {
    put_x(0, blockIdx.x, 0);
    put_g(0);
  }
  __syncthreads();
  // ---- accumulators ----
  f4v dw2[kR][2];
  float db2[kR];
#pragma unroll
  for (int i = 0; i < kR; ++i) {
    dw2[i][0] = dw2[i][1] = f4v{0.f, 0.f, 0.f, 0.f};
    db2[i] = 0.f;
  }
  f4v dw1[2][3];
#pragma unroll
  for (int b = 0; b < 2; ++b) dw1[b][0] = dw1[b][1] = dw1[b][2] = f4v{0.f, 0.f, 0.f, 0.f};
  float db1[2] = {0.f, 0.f}, dt0[2] = {0.f, 0.f}, dt1[2] = {0.f, 0.f};  // bias and temporal weights
  const float* w1l = W1L + hd * kHid * kW1L;

  // dZ from dH and H (registers, units x anchors), then the head's dX^T into
  // its slot dxs and dZ into transpose rows pub (either may be NULL)
  auto tail = [&](const f4v (&h)[2], const f4v (&dh)[2], float (*dxs)[kDXL], float (*pub)[kHB]) {
    f4v dz[2];
    if (hd == 4) {
#pragma unroll
      for (int e = 0; e < 8; ++e) dz[e >> 2][e & 3] = dh[e >> 2][e & 3] * (1.f - fexp(-h[e >> 2][e & 3]));
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) dz[e >> 2][e & 3] = h[e >> 2][e & 3] > 0.f ? dh[e >> 2][e & 3] : 0.f;
    }
    if (pub) {
#pragma unroll
      for (int b = 0; b < 2; ++b) *reinterpret_cast<f4v*>(&pub[fl][16 * b + 4 * fg]) = dz[b];
    }
    if (dxs) {
      // dX^T (inputs x anchors) = W1^T dZ^T, K = units
      f4v dx[3];
#pragma unroll
      for (int ct = 0; ct < 3; ++ct) dx[ct] = f4v{0.f, 0.f, 0.f, 0.f};
      // columns past 36 (lanes of the third block) give rows of dX^T that are not kept
      const int c2 = 32 + (fl & 3);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        float wr[4][3];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float* row = w1l + (16 * b + 4 * fg + r) * kW1L;
          wr[r][0] = row[fl];
          wr[r][1] = row[16 + fl];
          wr[r][2] = row[c2];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int ct = 0; ct < 3; ++ct) dx[ct] = mfma(wr[r][ct], dz[b][r], dx[ct]);
      }
      // lane (f, g) holds dX[anchor f][inputs 16 ct + 4 g + r]
#pragma unroll
      for (int ct = 0; ct < 3; ++ct)
        if (16 * ct + 4 * fg < kDXL) *reinterpret_cast<f4v*>(&dxs[fl][16 * ct + 4 * fg]) = dx[ct];
    }
  };
  // dW1 += dZ^T X, db1 += sum_a dZ, with dZ read by rows of anchors from the
  // transpose rows src of the wave that formed it; view: the item's
  auto acc_dw1 = [&](const float (*src)[kHB], const float (*xb)[kXL], int view) {
    float dzt[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) dzt[b][r] = src[4 * fg + r][16 * b + fl];
    float xa[3][4];
#pragma unroll
    for (int ct = 0; ct < 3; ++ct)
#pragma unroll
      for (int r = 0; r < 4; ++r) xa[ct][r] = xb[4 * fg + r][16 * ct + fl];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float c = (dzt[b][0] + dzt[b][1]) + (dzt[b][2] + dzt[b][3]);
      db1[b] += c;
      if (nx == 3) {
        dt0[b] = fmaf(dv.lt[view][0], c, dt0[b]);
        dt1[b] = fmaf(dv.lt[view][1], c, dt1[b]);
      }
      f4v p[3];
#pragma unroll
      for (int ct = 0; ct < 3; ++ct) p[ct] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int ct = 0; ct < 3; ++ct) p[ct] = mfma(dzt[b][r], xa[ct][r], p[ct]);
#pragma unroll
      for (int ct = 0; ct < 3; ++ct) dw1[b][ct] += p[ct];
    }
  };

  // ---- the running sums into the workgroup's partial of the parameter
  // gradients, four values of a lane at a time (their reads before the first
  // write) ----
  char* const P = reinterpret_cast<char*>(w.part + ((int64_t)blockIdx.x << 6));
  auto flush = [&](bool add) {
    int cl = fl, cg = fg;
    asm volatile("" : "+v"(cl), "+v"(cg));  // addresses are formed here, not held in registers over the items
    auto put4 = [&](const int (&pi)[4], const f4v& v, const bool (&ok)[4]) {
      uint32_t at[4];
      f4v old;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        at[e] = 4u * (((uint32_t)pi[e] >> 6) * ((uint32_t)w.nblk_w << 6) + ((uint32_t)pi[e] & 63u));
        old[e] = add && ok[e] ? *reinterpret_cast<const float*>(P + at[e]) : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ok[e]) *reinterpret_cast<float*>(P + at[e]) = old[e] + v[e];
    };
    auto over_groups = [&](float x) {  // sum over the four lane groups
      x += __shfl_xor(x, 16);
      return x + __shfl_xor(x, 32);
    };
#pragma unroll
    for (int i = 0; i < kR; ++i) {
      if (!active || i >= nt) break;
      const int r0 = 16 * (t0 + i);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        int pi[4];
        bool ok[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int o = r0 + 4 * cg + e;
          pi[e] = w2o + o * kHid + 16 * c + cl;
          ok[e] = o < rows;
        }
        put4(pi, dw2[i][c], ok);
        dw2[i][c] = f4v{0.f, 0.f, 0.f, 0.f};
      }
      const float sb = over_groups(db2[i]);
      put4({w2o + rows * kHid + r0 + cl, 0, 0, 0}, f4v{sb, 0.f, 0.f, 0.f},
           {cg == 0 && r0 + cl < rows, false, false, false});
      db2[i] = 0.f;
    }
    if (hw1 < 0) return;
    const int o1w = (int)ht.off[hw1], oxw = (int)ht.xoff[hw1];  // the head of this wave's dW1
    // extra input columns: the distance weight's gradient is column 35 of the
    // products with X; the temporal weights' gradients are the items' bias
    // gradients times their view's embedding
    const bool dist = cl == 3 && nx > 0, lt = cg == 0 && nx == 3;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int ct = 0; ct < 3; ++ct) {
        int pi[4];
        bool ok[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int u = 16 * b + 4 * cg + e;
          pi[e] = ct == 2 && dist ? oxw + u * nx : o1w + u * kIn + 16 * ct + cl;
          ok[e] = ct < 2 || cl < 3 || dist;
        }
        put4(pi, dw1[b][ct], ok);
        dw1[b][ct] = f4v{0.f, 0.f, 0.f, 0.f};
      }
      const float sb = over_groups(db1[b]), s0 = over_groups(dt0[b]), s1 = over_groups(dt1[b]);
      const int u = 16 * b + cl;
      put4({o1w + kHid * kIn + u, oxw + u * 3 + 1, oxw + u * 3 + 2, 0}, f4v{sb, s0, s1, 0.f}, {cg == 0, lt, lt, false});
      db1[b] = dt0[b] = dt1[b] = 0.f;
    }
  };
  f4v hp[2];  // the feature waves' H of the previous item
  hp[0] = hp[1] = f4v{0.f, 0.f, 0.f, 0.f};
  float gfeat = 0.f, gxyz = 0.f;  // anchor gradients of the tile, over its views
  int tile = blockIdx.x, view = 0, ptile = 0, pview = 0;  // this item's and the previous one's
  int xcur = 0, xprev = 2;                                // their input buffers
  bool have = tile < ngrid;
  const int chunk = kChainViews * ((ngrid - 1 - (int)blockIdx.x) / (int)gridDim.x + 1) + 1;
  int left = chunk;  // items until the running sums go into the partial
  bool add = false;  // the partial holds an earlier chunk's sums
  // item by item, and one more round for what the last item left
  for (int par = 0, prev = 0; have || prev; par ^= 1) {
    int ntile = tile, nview = view + 1;
    if (nview == V) {
      nview = 0;
      ntile += (int)gridDim.x;
    }
    const bool more = have && ntile < ngrid;
    const int xnext = xcur == 2 ? 0 : xcur + 1;
    if (more) {
      if (ntile != tile) fetch_x(ntile);
      fetch_g(ntile, nview);
    }
    f4v h[2];
    h[0] = h[1] = f4v{0.f, 0.f, 0.f, 0.f};
    if (have && active) {
      const float (*xb)[kXL] = XB[xcur];
      const float* gb = GB + par * C::kGB;
      const int nanch = A - tile * 16;  // anchors of the tile (or more)
      f4v dh[2];
      dh[0] = dh[1] = f4v{0.f, 0.f, 0.f, 0.f};
      // Z^T (units x anchors) = W1 X^T, K = inputs
      f4v z[2];
      z[0] = z[1] = f4v{0.f, 0.f, 0.f, 0.f};
      {
        // every operand requested before the first product
        float x[9], wa[9], wb[9];
#pragma unroll
        for (int s = 0; s < 9; ++s) {
          x[s] = xb[fl][4 * s + fg];
          wa[s] = w1l[fl * kW1L + 4 * s + fg];
          wb[s] = w1l[(16 + fl) * kW1L + 4 * s + fg];
        }
#pragma unroll
        for (int s = 0; s < 9; ++s) {
          z[0] = mfma(wa[s], x[s], z[0]);
          z[1] = mfma(wb[s], x[s], z[1]);
        }
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        f4v b1 = {b1r[b][0], b1r[b][1], b1r[b][2], b1r[b][3]};
        if (nx == 3) {
          // the view's temporal term
          const f4v s0 = *reinterpret_cast<const f4v*>(&TW[hd * kHid + 16 * b + 4 * fg]);
          const f4v s1 = *reinterpret_cast<const f4v*>(&TW[(kHeads + hd) * kHid + 16 * b + 4 * fg]);
#pragma unroll
          for (int r = 0; r < 4; ++r) b1[r] += s0[r] * dv.lt[view][0] + s1[r] * dv.lt[view][1];
        }
        z[b] += b1;
      }
      if (hd == 4) {
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e >> 2][e & 3] = fsoftplus(z[e >> 2][e & 3]);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e >> 2][e & 3] = fmaxf(z[e >> 2][e & 3], 0.f);
      }
      // H by rows of anchors (B operand of dW2)
#pragma unroll
      for (int b = 0; b < 2; ++b) *reinterpret_cast<f4v*>(&HBw[fl][16 * b + 4 * fg]) = h[b];
      wave_sync();
      float ht_[2][4];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) ht_[b][r] = HBw[4 * fg + r][16 * b + fl];
      wave_sync();
      // row tiles i0 .. i0 + cnt - 1 together, so that their product chains interleave
      auto row_tiles = [&](auto cnt, auto first) {
        constexpr int N = decltype(cnt)::value, i0 = decltype(first)::value;
        // Y (anchors x rows) = H W2^T, K = units
        f4v y[N], dy[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
          y[i] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int r = 0; r < 4; ++r) dy[i][r] = gb[goff[i0 + i] + (4 * fg + r) * k];  // a valid location for every lane
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < N; ++i) y[i] = mfma(h[b][r], w2y[i0 + i][b][r], y[i]);
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) dy[i][r] = rok[i0 + i] && 4 * fg + r < nanch ? dy[i][r] : 0.f;
        if (hd < 3) {
          // sigmoid outputs (scaled by l_s for the scale head); rotation and feature are raw
#pragma unroll
          for (int i = 0; i < N; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float s = fsigm(y[i][r] + b2r[i0 + i]);
              dy[i][r] *= hd == 2 ? dc.l_s * s * (1.f - s) : s * (1.f - s);
            }
        }
        // dY transposed through LDS
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) HBw[4 * fg + r][16 * i + fl] = dy[i][r];
        wave_sync();
        f4v dyt[N];
#pragma unroll
        for (int i = 0; i < N; ++i) dyt[i] = *reinterpret_cast<const f4v*>(&HBw[fl][16 * i + 4 * fg]);
        wave_sync();
        // dW2 (rows x units) += dY^T H, K = anchors
        f4v p[N][2];
#pragma unroll
        for (int i = 0; i < N; ++i) p[i][0] = p[i][1] = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int i = 0; i < N; ++i)
#pragma unroll
            for (int b = 0; b < 2; ++b) p[i][b] = mfma(dy[i][r], ht_[b][r], p[i][b]);
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int b = 0; b < 2; ++b) dw2[i0 + i][b] += p[i][b];
#pragma unroll
        for (int i = 0; i < N; ++i) db2[i0 + i] += (dy[i][0] + dy[i][1]) + (dy[i][2] + dy[i][3]);
        // dH^T (units x anchors) += W2^T dY^T, K = rows
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int b = 0; b < 2; ++b) dh[b] = mfma(w2h[i0 + i][b][r], dyt[i][r], dh[b]);
      };
      using I0 = std::integral_constant<int, 0>;
      using I1 = std::integral_constant<int, 1>;
      using I2 = std::integral_constant<int, 2>;
      if (nt >= 2) row_tiles(I2{}, I0{});
      else if (nt == 1) row_tiles(I1{}, I0{});
      if (nt == 3) row_tiles(I1{}, I2{});
      if constexpr (kR > 3)
        if (nt == 4) row_tiles(I2{}, I2{});
      if (wv < 4) {
        tail(h, dh, DX[xcur][wv], wv == 3 ? HR[par] : HBw);
        if (wv < 3) {
          wave_sync();
          acc_dw1(HBw, xb, view);
        }
      } else {
        // the feature waves' dH partials, summed below in a fixed order
#pragma unroll
        for (int b = 0; b < 2; ++b) *reinterpret_cast<f4v*>(&DH[((par * 4 + q) * 64 + lane) * 8 + 4 * b]) = dh[b];
      }
    }
    // ---- what the previous item left to other waves ----
    if (prev) {
      if (wv == 4) acc_dw1(HR[par ^ 1], XB[xprev], pview);  // the rotation head's dW1
      if (wv >= 6 && has_feat) {
        f4v dh[2];
        const float* D = DH + (par ^ 1) * 4 * 64 * 8;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const f4v p0 = *reinterpret_cast<const f4v*>(&D[(0 * 64 + lane) * 8 + 4 * b]);
          const f4v p1 = *reinterpret_cast<const f4v*>(&D[(1 * 64 + lane) * 8 + 4 * b]);
          const f4v p2 = *reinterpret_cast<const f4v*>(&D[(2 * 64 + lane) * 8 + 4 * b]);
          const f4v p3 = *reinterpret_cast<const f4v*>(&D[(3 * 64 + lane) * 8 + 4 * b]);
          dh[b] = (p0 + p1) + (p2 + p3);
        }
        // wave 6: dX; wave 7: dW1
        tail(hp, dh, wv == 6 ? DXF[par ^ 1] : nullptr, wv == 7 ? HBw : nullptr);
        if (wv == 7) {
          wave_sync();
          acc_dw1(HBw, XB[xprev], pview);
        }
      }
    }
    hp[0] = h[0];
    hp[1] = h[1];
    if (more) {
      put_x(xnext, ntile, nview);
      put_g(par ^ 1);
    }
    __syncthreads();  // the previous item's dX is complete; the next item's inputs are staged
    // ---- anchor gradients of the previous item ----
    if (prev) {
      const int a0 = ptile * 16, a = t >> 5, c = t & 31;
      const float (*D0)[16][kDXL] = DX[xprev];
      const float (*D4)[kDXL] = DXF[par ^ 1];
      const bool first = pview == 0, last = pview == V - 1;
      {
        float v = (D0[0][a][c] + D0[1][a][c]) + (D0[2][a][c] + D0[3][a][c]);
        if (has_feat) v += D4[a][c];
        gfeat = first ? v : gfeat + v;
        if (last && d_feat && a0 + a < A) d_feat[(int64_t)(a0 + a) * 32 + c] = gfeat;
      }
      if (wv == 0) {
        // lane 16 c + a: component c of anchor a; lanes 48 + a: its distance
        const int col = 32 + fg;
        float g = (D0[0][fl][col] + D0[1][fl][col]) + (D0[2][fl][col] + D0[3][fl][col]);
        if (has_feat) g += D4[fl][col];
        const float del = XB[xprev][fl][col], dist = XB[xprev][fl][36];
        const float pd = fg < 3 ? del * g : 0.f;
        const float p1 = pd + __shfl_xor(pd, 16);
        const float pr = p1 + __shfl_xor(p1, 32);
        const float gdist = nx > 0 ? __shfl(g, 48 + fl) : 0.f;
        // through delta = D / |D| (projected, scaled by 1/|D|) and |D| (along delta)
        const float dD = a0 + fl < A && fg < 3 ? (g - del * pr) / dist + gdist * del : 0.f;
        gxyz = first ? dD : gxyz + dD;
        if (last && d_xyz && a0 + fl < A && fg < 3) d_xyz[(int64_t)fg * A + a0 + fl] = gxyz;
        // the camera-centre sum over the anchors
        float x = dD;
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xF, 0xF, true));  // row_ror 8
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xF, 0xF, true));  // row_ror 4
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xF, 0xF, true));  // row_ror 2
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xF, 0xF, true));  // row_ror 1
        if (fl == 0 && fg < 3) DC[3 * pview + fg] -= x;
      }
    }
    if (--left == 0 || !have) {
      if (want_params) flush(add);
      add = true;
      left = chunk;
    }
    prev = have;
    ptile = tile;
    pview = view;
    xprev = xcur;
    xcur = xnext;
    tile = ntile;
    view = nview;
    have = more;
  }
  // ---- the workgroup's camera-centre partials ----
  __syncthreads();
  if (t < 3 * V) w.dcpart[(int64_t)blockIdx.x * 3 * V + t] = DC[t];
}

template <int kR>
void launch_k(const DecodeConst& dc, const HeadTable& ht, const DecodeViews& dv, const float* xyz, const float* feat,
              const float* params, const PlaneTable& pt, const DecWork& w, float* d_xyz,
              float* d_feat, bool want_params, hipStream_t s) {
  constexpr int kBytes = Lds<kR>::kFloats * (int)sizeof(float);
  static bool attr_set = false;  // more than 64 KiB of dynamic LDS
  if (!attr_set) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k_dec_bwd<kR>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, kBytes);
    attr_set = true;
  }
  hipLaunchKernelGGL(k_dec_bwd<kR>, dim3((unsigned)w.nblk_w), dim3(kBT), kBytes, s, dc, ht, dv,
                     xyz, feat, params, pt, w, d_xyz, d_feat, want_params ? 1 : 0);
}

}  // namespace

int64_t dec_bwd_blocks(int64_t n_anchors) {
  const int64_t tiles = (n_anchors + 15) / 16;
  return tiles < kMaxWG ? tiles : kMaxWG;
}

void launch_dec_bwd(const DecodeConst& dc, const HeadTable& ht, const DecodeViews& dv, const float* xyz,
                    const float* feat, const float* params, const asgs_gaussians& dg, const DecWork& w,
                    float* d_xyz, float* d_feat, bool want_params, hipStream_t s) {
  const PlaneTable pt = plane_table(dc, ht, dg);
  // second-layer row tiles per wave: the rotation head has ceil(4 k / 16),
  // each feature wave ceil(k / 4)
  if (dc.k <= 12)
    launch_k<3>(dc, ht, dv, xyz, feat, params, pt, w, d_xyz, d_feat, want_params, s);
  else
    launch_k<4>(dc, ht, dv, xyz, feat, params, pt, w, d_xyz, d_feat, want_params, s);
}

}  // namespace asgs
