// MFMA GEMMs y = X W^T for the expert's projections.  No workgroup ever
// waits on another: an output tile is reduced inside one workgroup, or written
// as a split-K partial that a later launch adds up (on this 8-XCD part an
// agent-scope fence writes back and invalidates the XCD's whole L2, so
// in-kernel cross-workgroup reductions cost far more than a launch).
//
// gemm_skinny -- the per-step projections: row-major operands up to
//   kSkinnyRows token rows, tiled ones of any number where the planner's cost
//   is below gemm_tile's (the caller decides both, and sees to it that X stays
//   below 2 GiB: its loads have 32-bit offsets).
//   A workgroup of 8 waves owns 16*NSUB rows of W (NSUB = 2: a gate/up pair
//   of interleaved 16-row blocks), 16*MS token rows and one K-range
//   (split-K across workgroups only where the epilogue writes partials).  The
//   range's k-steps (64 bytes of a row) are spread evenly over the waves.
//   Every operand goes straight from global memory into MFMA-layout
//   registers: a round issues all W and X loads of the wave before the first
//   MFMA, so a workgroup pays one memory latency per round instead of one per
//   staging step.  The eight partial tiles are summed in wave order through
//   LDS and waves 0..MS-1 run the epilogue of one 16-row subtile each.
//   What bounds it is the bytes a compute unit takes in (about 48 GB/s) and
//   the fixed latency of a launch, so the tile is the one that spreads the
//   least bytes over 256 compute units (skinny_cost).  In a chain of cold
//   weights, against tiles that always hold every token row with branchy loads
//   in 128-wide chunks (50 rows, bf16): 960 x 720 5.7 -> 3.6 us, 1600 x 720
//   5.8 -> 3.9, gate/up 4096 x 720 6.2 -> 4.8 (row-major operands: 3.8, 4.2, 5.2),
//   down 720 x 2048 4.7 -> 3.5; 51 rows, 8192 x 1024 9.4 -> 7.2.
//
// gemm_wide -- fp32 with M > 128.  Four waves along N (NT = 64*NSUB), X
//   staged per K-slice in LDS and shared by the four waves, K-slices looped
//   inside the workgroup.
//
// gemm_tile -- bf16 with M > 128 (batched requests, the prefix K/V build),
//   where LDS bandwidth and the MFMAs bound the work.  Eight waves (2 x 4) own
//   a (16*MR) x (32*NS) output tile; slices of 64 k-values of X and W stream
//   into a ring of LDS stages by direct-to-LDS loads, several slices ahead of
//   the MFMAs, and the epilogue stores from the accumulators.  A K that is not
//   a multiple of 64 takes gemm_tile_rs instead: four waves (2 x 2), the next
//   slice's loads held in registers during the MFMAs, padded LDS rows.  Tiles
//   along M are numbered fastest and blocks are renumbered so that consecutive
//   tiles (which share one W slice) run on the same XCD and its L2.
//
// Operand layout: in a chunk, lane l of a wave reads 16-byte vector v of row
// (l % 16) at k-offset v*4*E + (l/16)*E, for W and X alike, so the MFMA's k
// order is a permutation common to both operands and every load instruction
// of a wave reads 64 contiguous bytes per row.
#include <algorithm>
#include <cmath>
#include <utility>

#include "gemm_epilogue.h"

namespace {

constexpr int VPL = 4;   // 16-byte vectors per lane per chunk
constexpr int WKS = 8;   // waves of a skinny workgroup

// Stage X rows m0 .. m0+MT-1, columns k0 .. k0+KW-1 (KW a multiple of E) into
// LDS with row pitch `pitch` elements; zeros outside [M] x [K].  A thread
// issues the loads of up to UB items before storing any of them.
template <typename T, int MT>
VLA_DEV void stage_x(const GemmArgs& a, T* xs, int pitch, int m0, int k0, int KW) {
  constexpr int E = ElemTraits<T>::E;
  constexpr int UB = 8;
  const int vrow = KW / E;
  const int total = MT * vrow;
  const int nthr = blockDim.x;
  const T* X = reinterpret_cast<const T*>(a.X);
  for (int base = threadIdx.x; base < total; base += UB * nthr) {
    uint4 v[UB];
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int i = base + u * nthr;
      const int row = i / vrow, kv = i - row * vrow;
      const bool ok = i < total && (m0 + row) < a.M && (k0 + kv * E) < a.K;
      v[u] = ok ? ldg16(X + act_off<T>(m0 + row, k0 + kv * E, a.ldx, a.xt)) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int i = base + u * nthr;
      if (i < total) {
        const int row = i / vrow, kv = i - row * vrow;
        *reinterpret_cast<uint4*>(xs + (size_t)row * pitch + kv * E) = v[u];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// NV: k-steps (4 E values: one 16-byte vector per lane group) of one wave and
// round.  TL: both operands tiled (device_common.h): every load is one whole
// kilobyte at a wave-uniform offset; padding reads the zeros stored there.
template <typename T, int MS, int NSUB, int NV, bool TL>
__global__ __launch_bounds__(64 * WKS) void gemm_skinny(GemmArgs a) {
  constexpr int E = ElemTraits<T>::E;
  constexpr int KSTEP = 4 * E;         // k-values of one step: one vector per lane group
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4* red = reinterpret_cast<f32x4*>(smem);  // [WKS][MS][NSUB][64]

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, g4 = lane >> 4;
  // grid (8, row tiles, columns / 8): workgroups go round robin over the XCDs
  // in the x index, so every row tile of a W tile runs on one XCD and its L2
  // reads that tile's weights from memory once
  const int col = blockIdx.z * 8 + blockIdx.x;
  const int split = col & (a.nsplit - 1), ntile = col >> a.split_log2;
  if (ntile >= a.n_tiles) return;
  const int m0 = blockIdx.y * 16 * MS;
  const int nb = ntile * 16 * NSUB;
  const int k0 = split * a.kper;
  const int k1 = min(a.K, k0 + a.kper);
  // Buffer loads over the workgroup's own rows: rows past M or N are past the
  // buffer's end and read zero, so a row costs no branch.
  const rsrc_t W = TL ? make_rsrc(reinterpret_cast<const T*>(a.W) + (size_t)(nb >> 4) * a.wt * (16 * KSTEP),
                                  (unsigned)min((a.N - nb + 15) >> 4, NSUB) * (unsigned)a.wt * 1024u)
                      : make_rsrc(reinterpret_cast<const T*>(a.W) + (size_t)nb * a.K,
                                  (unsigned)min(a.N - nb, 16 * NSUB) * (unsigned)a.K * (unsigned)sizeof(T));
  const rsrc_t X = TL ? make_rsrc(a.X, (unsigned)a.wt * (unsigned)a.xt * 64u)
                      : make_rsrc(reinterpret_cast<const T*>(a.X) + (size_t)m0 * a.ldx,
                                  ((unsigned)(min(a.M - m0, 16 * MS) - 1) * (unsigned)a.ldx + (unsigned)a.K) * (unsigned)sizeof(T));

  f32x4 acc[MS][NSUB];
#pragma unroll
  for (int ms = 0; ms < MS; ++ms)
#pragma unroll
    for (int s = 0; s < NSUB; ++s) acc[ms][s] = f32x4{0.f, 0.f, 0.f, 0.f};

  // wave w takes steps w NV .. of every round of WKS NV steps; a wave without
  // steps loads nothing (an out-of-range load costs the address unit as much
  // as any other)
  for (int kr = k0 + wave * NV * KSTEP; kr < k1; kr += WKS * NV * KSTEP) {
    uint4 wreg[NSUB][NV], xreg[MS][NV];
    const int kl = kr + g4 * E;
    if constexpr (TL) {
      // a step past the range (the last wave's) or a subtile past N loads
      // zeros from past the buffer's end, and no row of X past the padded ones
      // is read
      const unsigned lo = (unsigned)(r16 * 64 + g4 * 16), kb = (unsigned)(kr / KSTEP), ke = (unsigned)((k1 + KSTEP - 1) / KSTEP);
      const int subs = min((a.N - nb + 15) >> 4, NSUB);
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int s = 0; s < NSUB; ++s) {
          const TileLoad at = skinny_w_at(lo, s, subs, kb + v, ke, a.wt);
          wreg[s][v] = buf_ld16(W, at.lane, at.uni);
        }
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int ms = 0; ms < MS; ++ms) {
          const TileLoad at = skinny_x_at(lo, m0 + ms * 16, a.xt, kb + v, ke);
          xreg[ms][v] = buf_ld16(X, at.lane, at.uni);
        }
    } else {
    unsigned wo[NSUB], xo[MS];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) wo[s] = (unsigned)((s * 16 + r16) * a.K + kl) * (unsigned)sizeof(T);
#pragma unroll
    for (int ms = 0; ms < MS; ++ms) xo[ms] = (unsigned)((ms * 16 + r16) * a.ldx + kl) * (unsigned)sizeof(T);
    if (kr + NV * KSTEP <= k1) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int v = 0; v < NV; ++v) wreg[s][v] = buf_ld16(W, wo[s] + 64u * v);
#pragma unroll
      for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int v = 0; v < NV; ++v) xreg[ms][v] = buf_ld16(X, xo[ms] + 64u * v);
    } else {   // the range's end: vectors past it read zero
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int v = 0; v < NV; ++v) wreg[s][v] = buf_ld16(W, kl + v * KSTEP < k1 ? wo[s] + 64u * v : kOob);
#pragma unroll
      for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int v = 0; v < NV; ++v) xreg[ms][v] = buf_ld16(X, kl + v * KSTEP < k1 ? xo[ms] + 64u * v : kOob);
    }
    }
    __builtin_amdgcn_sched_barrier(0);   // every load of the round in flight before the first MFMA
#pragma unroll
    for (int ms = 0; ms < MS; ++ms)
#pragma unroll
      for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int v = 0; v < NV; ++v) mma16(acc[ms][s], xreg[ms][v], wreg[s][v], T());
  }

  // sum the eight partial tiles in wave order; wave ms < MS finishes subtile ms
#pragma unroll
  for (int ms = 0; ms < MS; ++ms)
#pragma unroll
    for (int s = 0; s < NSUB; ++s) red[((wave * MS + ms) * NSUB + s) * 64 + lane] = acc[ms][s];
  __syncthreads();
  if (wave >= MS) return;
  f32x4 r[1][NSUB];
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    r[0][s] = red[((0 * MS + wave) * NSUB + s) * 64 + lane];
#pragma unroll
    for (int w = 1; w < WKS; ++w) r[0][s] += red[((w * MS + wave) * NSUB + s) * 64 + lane];
  }
  wave_epilogue<T, 1, NSUB>(a, r, m0 + wave * 16, nb, split);
}

// ---------------------------------------------------------------------------
template <typename T, int MS, int NSUB, int NC>
__global__ __launch_bounds__(256) void gemm_wide(GemmArgs a) {
  constexpr int E = ElemTraits<T>::E;
  constexpr int KCL = VPL * E;
  constexpr int KC = 4 * KCL;
  constexpr int KS = NC * KC;
  constexpr int MT = 16 * MS;
  constexpr int NT = 64 * NSUB;
  constexpr int PITCH = KS + E;
  extern __shared__ __align__(16) unsigned char smem[];
  T* xs = reinterpret_cast<T*>(smem);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, g4 = lane >> 4;
  const int N = a.N, K = a.K;
  const int ntile = blockIdx.x % a.n_tiles, mtile = blockIdx.x / a.n_tiles;
  const int m0 = mtile * MT;
  const int nb = ntile * NT + wave * 16 * NSUB;
  const T* W = reinterpret_cast<const T*>(a.W);

  f32x4 acc[MS][NSUB];
#pragma unroll
  for (int ms = 0; ms < MS; ++ms)
#pragma unroll
    for (int s = 0; s < NSUB; ++s) acc[ms][s] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int k0 = 0; k0 < K; k0 += KS) {
    uint4 wreg[NSUB][NC][VPL];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int n = nb + s * 16 + r16;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int v = 0; v < VPL; ++v) {
          const int k = k0 + c * KC + g4 * KCL + v * E;
          wreg[s][c][v] = (n < N && k < K) ? ldg16(W + (a.wt ? wtile_off<T>(n, k, a.wt) : (size_t)n * K + k))
                                           : make_uint4(0, 0, 0, 0);
        }
    }
    if (k0 > 0) __syncthreads();  // previous slice's LDS reads done
    stage_x<T, MT>(a, xs, PITCH, m0, k0, KS);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (k0 + c * KC >= K) break;
#pragma unroll
      for (int ms = 0; ms < MS; ++ms) {
        const T* xrow = xs + (size_t)(ms * 16 + r16) * PITCH + c * KC + g4 * KCL;
        uint4 xf[VPL];
#pragma unroll
        for (int v = 0; v < VPL; ++v) xf[v] = *reinterpret_cast<const uint4*>(xrow + v * E);
#pragma unroll
        for (int s = 0; s < NSUB; ++s)
#pragma unroll
          for (int v = 0; v < VPL; ++v) mma16(acc[ms][s], xf[v], wreg[s][c][v], T());
      }
    }
  }
  wave_epilogue<T, MS, NSUB>(a, acc, m0, nb, 0);
}


// ---------------------------------------------------------------------------
constexpr int TBK = 64;           // K-slice of gemm_tile
constexpr int TPITCH = TBK + 8;   // LDS row pitch in elements (16 bytes of padding)

// LDS of gemm_tile_rs: two K-slice buffers of X and W rows.
template <int MS, int NS>
constexpr size_t tile_lds_bytes() {
  return (size_t)2 * (32 * MS + 32 * NS) * TPITCH * sizeof(bf16_t);
}

// Epilogue of the tiled kernels, straight from the accumulators.  W is the
// MFMA's row operand, so a lane holds four consecutive columns n of one token
// row m (for EPI_GLU four of a gate and of its up subtile) and writes them
// with one 8- or 16-byte store; a row's 16 columns are four lanes' stores.
VLA_DEV void store4(float* p, f32x4 v, bool vec) {
  if (vec) *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  else { p[0] = v[0]; p[1] = v[1]; p[2] = v[2]; p[3] = v[3]; }
}
VLA_DEV void store4(bf16_t* p, f32x4 v, bool vec) {
  if (vec) *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
  else { p[0] = f2bf(v[0]); p[1] = f2bf(v[1]); p[2] = f2bf(v[2]); p[3] = f2bf(v[3]); }
}
// Columns n .. n+3 of which only the first `nv` exist.
template <typename T>
VLA_DEV void store4n(T* p, f32x4 v, int nv, bool vec) {
  if (nv >= 4) { store4(p, v, vec); return; }
  for (int j = 0; j < nv; ++j) {
    if constexpr (sizeof(T) == 4) p[j] = v[j]; else p[j] = f2bf(v[j]);
  }
}
VLA_DEV f32x4 act4(int act, f32x4 v) { return f32x4{act_f(act, v[0]), act_f(act, v[1]), act_f(act, v[2]), act_f(act, v[3])}; }

// acc[ms][ns]: rows mb + 16 ms + r16, columns nb + 16 ns + 4 g4 + i.
// msn: row subtiles of this wave (MSW, or one less).
template <int MSW, int NSW>
VLA_DEV void tile_epilogue(const GemmArgs& a, const f32x4 (&acc)[MSW][NSW], int mb, int nb, int split, int msn = MSW) {
  const int lane = threadIdx.x & 63, r16 = lane & 15, c0 = (lane >> 4) * 4;
  const int M = a.M, N = a.N;
  // f(m, n, nv, v) for every 4-column group that exists
  auto each = [&](auto&& f) {
#pragma unroll
    for (int ms = 0; ms < MSW; ++ms) {
      const int m = mb + 16 * ms + r16;
      if (ms >= msn || m >= M) continue;
#pragma unroll
      for (int ns = 0; ns < NSW; ++ns) {
        const int n = nb + 16 * ns + c0;
        if (n < N) f(m, n, N - n, acc[ms][ns]);
      }
    }
  };
  switch (a.epi) {
    case EPI_GLU: {
      const bool vec = (a.ldo & 3) == 0;
      const int act = a.act, F = N / 2;
#pragma unroll
      for (int ms = 0; ms < MSW; ++ms) {
        const int m = mb + 16 * ms + r16;
        if (ms >= msn || m >= M) continue;
#pragma unroll
        for (int j = 0; j < NSW / 2; ++j) {
          const int fc = nb / 2 + 16 * j + c0;
          if (fc >= F) continue;
          const f32x4 h = act4(act, acc[ms][2 * j]) * acc[ms][2 * j + 1];
          if (a.out_f32) store4n(reinterpret_cast<float*>(a.out) + (size_t)m * a.ldo + fc, h, F - fc, vec);
          else store4n(reinterpret_cast<bf16_t*>(a.out) + act_off<bf16_t>(m, fc, a.ldo, a.ot), h, F - fc, vec);
        }
      }
      break;
    }
    case EPI_STORE: {
      const bool vec = (a.ldo & 3) == 0;
      each([&](int m, int n, int nv, f32x4 v) {
        if (a.bias)
          v += f32x4{a.bias[n], nv > 1 ? a.bias[n + 1] : 0.f, nv > 2 ? a.bias[n + 2] : 0.f, nv > 3 ? a.bias[n + 3] : 0.f};
        v = act4(a.act, v);
        if (a.out_f32) store4n(reinterpret_cast<float*>(a.out) + (size_t)m * a.ldo + n, v, nv, vec);
        else store4n(reinterpret_cast<bf16_t*>(a.out) + act_off<bf16_t>(m, n, a.ldo, a.ot), v, nv, vec);
      });
      break;
    }
    case EPI_PARTIAL: {
      float* out = reinterpret_cast<float*>(a.out) + (size_t)split * M * a.ldo;
      const bool vec = (a.ldo & 3) == 0;
      each([&](int m, int n, int nv, f32x4 v) { store4n(out + (size_t)m * a.ldo + n, v, nv, vec); });
      break;
    }
    case EPI_RESID: {
      const bool vec = (a.ldxr & 3) == 0;
      each([&](int m, int n, int nv, f32x4 v) {
        float* xp = a.xres + (size_t)m * a.ldxr + n;
        if (vec && nv >= 4) {
          const float4 x = *reinterpret_cast<const float4*>(xp), al = *reinterpret_cast<const float4*>(a.alpha + n);
          *reinterpret_cast<float4*>(xp) = make_float4(x.x + al.x * v[0], x.y + al.y * v[1], x.z + al.z * v[2], x.w + al.w * v[3]);
        } else {
          for (int j = 0; j < 4 && j < nv; ++j) xp[j] = xp[j] + a.alpha[n + j] * v[j];
        }
      });
      break;
    }
    case EPI_KVCACHE: {
      const int G = a.d_kv / a.hd;
      each([&](int m, int n, int nv, f32x4 v) {
        // hd, d_kv and lay_cols are multiples of 16: the four columns share a head's row
        const int b = m / a.P, p = m - b * a.P;
        const int slot = a.lay_cols > 0 ? n / a.lay_cols : 0;
        const int nl = n - slot * a.lay_cols;
        const int kv = nl / a.d_kv, rem = nl - kv * a.d_kv;
        const int g = rem / a.hd, cc = rem - g * a.hd;
        const size_t o = (size_t)slot * a.lay_stride + ((((size_t)kv * a.B + b) * G + g) * a.P + p) * a.hd + cc;
        store4n(reinterpret_cast<bf16_t*>(a.cache) + o, v, nv, true);
      });
      break;
    }
    case EPI_EULER: {
      const CallParams* cp = a.cp;
      const float dt = cp->tau[a.step + 1] - cp->tau[a.step];
      each([&](int m, int n, int nv, f32x4 v) {
        const int t = a.stok ? m % a.stok : 1;   // state-token rows: no action
        const int am = a.stok ? (m / a.stok) * (a.stok - 1) + t - 1 : m;
        if (t == 0) return;
        for (int j = 0; j < 4 && j < nv; ++j) {
          const int nn = n + j;
          const float vv = v[j] + a.bias[nn];
          float* ap = a.a + (size_t)am * N + nn;
          const float an = a.regression ? vv : (*ap + dt * vv);
          *ap = an;
          if (a.last) {
            float o = an;
            if (cp->act_std) o *= cp->act_std[nn];
            if (cp->act_mean) o += cp->act_mean[nn];
            cp->actions_out[(size_t)am * N + nn] = o;
          }
        }
      });
      break;
    }
    default:
      break;
  }
}

template <int MS, int NS>
__global__ __launch_bounds__(256) void gemm_tile_rs(GemmArgs a) {
  constexpr int BM = 32 * MS, BN = 32 * NS, ROWS = BM + BN;
  constexpr int LPT = ROWS * (TBK / 8) / 256;  // 16-byte loads per thread and slice
  constexpr int XL = BM / 32;                  // of which X rows
  static_assert(ROWS % 32 == 0 && LPT * 256 == ROWS * (TBK / 8), "tile rows");
  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* lds = reinterpret_cast<bf16_t*>(smem);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, g4 = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int M = a.M, N = a.N, K = a.K;
  // consecutive workgroups go to consecutive XCDs: unit u runs on XCD u / per
  const int per = gridDim.x >> 3;
  const int u = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int tiles = a.m_tiles * a.n_tiles;
  if (u >= tiles * a.nsplit) return;
  const int split = u / tiles, t = u - split * tiles;
  const int ntile = t / a.m_tiles, mtile = t - ntile * a.m_tiles;
  const int m0 = mtile * BM, n0 = ntile * BN;
  const int k0 = split * a.kper;
  const int k1 = min(K, k0 + a.kper);

  // this thread's rows: chunk ch of tile rows (tid >> 3) + 32 i
  const int ch = tid & 7;
  const bf16_t* src[LPT];
  bool rok[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int row = (tid >> 3) + 32 * i;
    if (i < XL) {
      const int m = m0 + row;
      rok[i] = m < M;
      src[i] = reinterpret_cast<const bf16_t*>(a.X) + (size_t)(rok[i] ? m : 0) * a.ldx + ch * 8;
    } else {
      const int n = n0 + row - BM;
      rok[i] = n < N;
      src[i] = reinterpret_cast<const bf16_t*>(a.W) + (size_t)(rok[i] ? n : 0) * K + ch * 8;
    }
  }
  uint4 pre[LPT];
  auto gload = [&](int kb) {
    const bool kok = kb + ch * 8 < k1;
#pragma unroll
    for (int i = 0; i < LPT; ++i) pre[i] = (rok[i] && kok) ? ldg16(src[i] + kb) : make_uint4(0, 0, 0, 0);
  };
  auto lstore = [&](int buf) {
    bf16_t* b = lds + (size_t)buf * ROWS * TPITCH;
#pragma unroll
    for (int i = 0; i < LPT; ++i)
      *reinterpret_cast<uint4*>(b + ((tid >> 3) + 32 * i) * TPITCH + ch * 8) = pre[i];
  };

  f32x4 acc[MS][NS];
#pragma unroll
  for (int ms = 0; ms < MS; ++ms)
#pragma unroll
    for (int ns = 0; ns < NS; ++ns) acc[ms][ns] = f32x4{0.f, 0.f, 0.f, 0.f};

  gload(k0);
  lstore(0);
  __syncthreads();
  int buf = 0;
  for (int kb = k0; kb < k1; kb += TBK) {
    const bool more = kb + TBK < k1;
    if (more) gload(kb + TBK);
    const bf16_t* lb = lds + (size_t)buf * ROWS * TPITCH;
#pragma unroll
    for (int kk = 0; kk < TBK / 32; ++kk) {
      uint4 af[MS], bq[NS];
#pragma unroll
      for (int ms = 0; ms < MS; ++ms)
        af[ms] = *reinterpret_cast<const uint4*>(lb + (wm * 16 * MS + ms * 16 + r16) * TPITCH + kk * 32 + g4 * 8);
#pragma unroll
      for (int ns = 0; ns < NS; ++ns)
        bq[ns] = *reinterpret_cast<const uint4*>(lb + (BM + wn * 16 * NS + ns * 16 + r16) * TPITCH + kk * 32 + g4 * 8);
#pragma unroll
      for (int ms = 0; ms < MS; ++ms)
#pragma unroll
        for (int ns = 0; ns < NS; ++ns) mma16(acc[ms][ns], bq[ns], af[ms], bf16_t());   // W rows x token rows
    }
    if (more) lstore(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }

  tile_epilogue<MS, NS>(a, acc, m0 + wm * 16 * MS, n0 + wn * 16 * NS, split);
}


// ---------------------------------------------------------------------------
// gemm_tile: the K-slices stream into a ring of NST LDS stages with
// direct-to-LDS loads (global_load_lds_dwordx4), NST - 1 slices ahead of the
// MFMAs, so several slices' latency overlaps without holding their bytes in
// registers.  A stage holds ROWS rows of 64 k-values (128 bytes); a load
// instruction of a wave fills 1 KB (eight rows), lane l writing row l/8,
// 16-byte slot l%8, and fetching the row's k-chunk (l%8) ^ (row%8): the XOR
// swizzle puts the eight rows one MFMA operand load reads into eight
// different bank groups.  Stages are separate LDS arrays indexed at compile
// time, so the compiler can tell the stage being read from the ones still in
// flight and does not wait for those.  Requires K % 64 == 0 (rows beyond M
// or N are loaded from a valid row and never stored).
//
// NWV = 8 waves, 2 x 4 (two per SIMD).  Every wave sums its
// outputs' k-products slice by slice in the same order, so the tile does not
// change a result.  The 256 x 256 tile (128 x 64 per
// wave) feeds 128 FLOP per staged byte instead of 85 (256 x 128); its two
// 64 KB stages fill the LDS, and a slice's MFMAs cover the next slice's load.
//
// The tile's height is any number MR of 16-row subtiles: the first row of
// waves takes the larger half, and the waves of one SIMD are one of each row,
// so an odd MR loads the four SIMDs evenly.  A height that divides the rows
// well saves the work of padding: 816 rows in four 208-row tiles instead of
// four of 256, 1600 in eight instead of seven that fill fewer compute units.
// 160 and 208 are the two heights between the powers of two that were built
// and measured; the planner weighs every tile by its cost, so a row count that
// neither divides well takes the one with the least padding and rounds.
template <int MR, int NS, int NWV>
struct Ring {
  static constexpr int BM = 16 * MR, BN = 32 * NS, ROWS = BM + BN;
  static constexpr int NST = ROWS <= 256 ? 4 : (ROWS <= 384 ? 3 : 2);   // stages (LDS <= 144 KB)
  static constexpr int NLD = ROWS / 8;                  // load instructions of the workgroup per slice (8 rows each)
  static constexpr int LPT = (NLD + NWV - 1) / NWV;     // at most, of one wave
  static constexpr int LASTW = NLD - (LPT - 1) * NWV;   // waves that issue the last one
  static constexpr int SB = ROWS * 8;                   // 16-byte slots per stage
  // rows of fp32 partials per epilogue pass through stage 0
  static constexpr int RP = (64 * (BN + 4) * 4 <= SB * 16) ? 64 : (32 * (BN + 4) * 4 <= SB * 16 ? 32 : 16);
};

template <int MR, int NS, int NWV>
__global__ __launch_bounds__(64 * NWV) void gemm_tile(GemmArgs a) {
  using R = Ring<MR, NS, NWV>;
  constexpr int BM = R::BM, BN = R::BN, NST = R::NST, LPT = R::LPT, SB = R::SB, D = NST - 1;
  constexpr int WN = NWV / 2;                          // waves along N (2 along M)
  constexpr int MSW = (MR + 1) / 2, NSW = BN / (16 * WN);   // most 16-row / all 16-column subtiles of a wave
  __shared__ v4u st0[SB], st1[SB], st2[NST > 2 ? SB : 1], st3[NST > 3 ? SB : 1];
  auto stage = [&](auto j) -> v4u* {
    constexpr int J = decltype(j)::value;
    if constexpr (J == 0) return st0;
    else if constexpr (J == 1) return st1;
    else if constexpr (J == 2) return st2;
    else return st3;
  };

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane & 15, g4 = lane >> 4;
  const int wm = __builtin_amdgcn_readfirstlane(wave / WN), wn = wave % WN;
  const int msn = MR % 2 && wm ? MSW - 1 : MSW;   // this wave's row subtiles
  const int M = a.M, N = a.N, K = a.K;
  const int per = gridDim.x >> 3;
  const int u = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  const int tiles = a.m_tiles * a.n_tiles;
  if (u >= tiles * a.nsplit) return;
  const int split = u / tiles, t = u - split * tiles;
  const int ntile = t / a.m_tiles, mtile = t - ntile * a.m_tiles;
  const int m0 = mtile * BM, n0 = ntile * BN;
  const int k0 = split * a.kper;
  const int nsl = (min(K, k0 + a.kper) - k0) / 64;

  // source of this lane's slot in load instruction i: row (i*NWV + wave)*8 + lane/8
  // elements from a slice to the next: 64 columns, or two k-tiles
  const size_t wstep = a.wt ? 1024 : 64, xstep = a.xt ? (size_t)64 * a.xt : 64;
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  const bf16_t* src[LPT];
  size_t step[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int row = (i * NWV + wave) * 8 + (lane >> 3);
    const int chunk = (lane & 7) ^ (row & 7);
    const bool isx = (i * NWV + wv) * 8 < BM;   // BM % 8 == 0: an instruction holds X rows or W rows
    step[i] = isx ? xstep : wstep;
    if (isx) {
      const int m = min(m0 + row, M - 1);
      src[i] = reinterpret_cast<const bf16_t*>(a.X) + act_off<bf16_t>(m, k0 + chunk * 8, a.ldx, a.xt);
    } else {
      const int n = min(n0 + row - BM, N - 1);
      src[i] = reinterpret_cast<const bf16_t*>(a.W) +
               (a.wt ? wtile_off<bf16_t>(n, k0 + chunk * 8, a.wt) : (size_t)n * K + k0 + chunk * 8);
    }
  }
  const bool last_ld = R::LASTW == NWV || wv < R::LASTW;   // this wave issues LPT loads a slice, else LPT - 1
  auto issue = [&](auto j, int sl) {
    v4u* b = stage(j);
#pragma unroll
    for (int i = 0; i < LPT; ++i)
      if (i + 1 < LPT || last_ld) dma16(src[i] + sl * step[i], b + (i * NWV + wave) * 64);
  };

  f32x4 acc[MSW][NSW];
#pragma unroll
  for (int ms = 0; ms < MSW; ++ms)
#pragma unroll
    for (int ns = 0; ns < NSW; ++ns) acc[ms][ns] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Operand rows of this lane and their swizzled slot for logical chunk c.
  // One k-half at a time keeps the registers under the two-wave limit; the
  // other wave of the SIMD hides the LDS latency.
  auto compute = [&](const v4u* b) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      v4u af[MSW], bq[NSW];
      const int c = kk * 4 + g4;
#pragma unroll
      for (int ms = 0; ms < MSW; ++ms) {
        const int row = wm * 16 * MSW + ms * 16 + r16;
        if (MR % 2 == 0 || ms + 1 < MSW || msn == MSW) af[ms] = b[row * 8 + (c ^ (row & 7))];
      }
#pragma unroll
      for (int ns = 0; ns < NSW; ++ns) {
        const int row = BM + wn * 16 * NSW + ns * 16 + r16;
        bq[ns] = b[row * 8 + (c ^ (row & 7))];
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ms = 0; ms < MSW; ++ms) {
        if (MR % 2 && ms + 1 == MSW && msn < MSW) continue;
#pragma unroll
        for (int ns = 0; ns < NSW; ++ns)
          acc[ms][ns] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, bq[ns]),
                                                                __builtin_bit_cast(bf16x8_t, af[ms]), acc[ms][ns],
                                                                0, 0, 0);
      }
    }
  };

  // prologue: slices 0 .. D-1 in flight
  [&]<int... J>(std::integer_sequence<int, J...>) {
    ((J < nsl ? issue(std::integral_constant<int, J>{}, J) : void()), ...);
  }(std::make_integer_sequence<int, D>{});

  for (int it0 = 0; it0 < nsl; it0 += NST) {
    [&]<int... J>(std::integer_sequence<int, J...>) {
      (
          [&] {
            const int it = it0 + J;
            if (it >= nsl) return;
            // slice `it` has landed once at most the D-1 later slices are pending
            if (it + D - 1 < nsl) {
              if (last_ld) __builtin_amdgcn_s_waitcnt(vm_wait((D - 1) * LPT));
              else __builtin_amdgcn_s_waitcnt(vm_wait((D - 1) * (LPT - 1)));
            } else {
              __builtin_amdgcn_s_waitcnt(vm_wait(0));
            }
            lds_barrier();
            // the stage of slice it-1 is free: refill it with slice it+D
            if (it + D < nsl) issue(std::integral_constant<int, (J + D) % NST>{}, it + D);
            compute(stage(std::integral_constant<int, J>{}));
          }(),
          ...);
    }(std::make_integer_sequence<int, NST>{});
  }
  if (a.epi != EPI_PARTIAL) {
    tile_epilogue<MSW, NSW>(a, acc, m0 + wm * 16 * MSW, n0 + wn * 16 * NSW, split, msn);
    return;
  }
  // Split-K partials, fp32: through LDS in passes of RP rows, so that whole
  // rows of the tile are written at once (a split tile is short, and its
  // partials are most of what it moves: 400 x 720 from K = 960 in three
  // splits 7.2 us this way, 8.8 with the accumulators' own 64-byte pieces).
  constexpr int RP = R::RP, CP = BN + 4, TPR = BN / 4;
  float* ct = reinterpret_cast<float*>(st0);
  float* out = reinterpret_cast<float*>(a.out) + (size_t)split * M * a.ldo;
  const bool vec = (a.ldo & 3) == 0;
  __builtin_amdgcn_s_waitcnt(vm_wait(0));
  lds_barrier();   // every wave is past its operand reads of stage 0
#pragma unroll
  for (int p = 0; p < (BM + RP - 1) / RP; ++p) {
#pragma unroll
    for (int ms = 0; ms < MSW; ++ms) {
      const int rb = wm * 16 * MSW + ms * 16;  // first row of subtile ms
      if (rb / RP == p && ms < msn) {
#pragma unroll
        for (int ns = 0; ns < NSW; ++ns)
          *reinterpret_cast<f32x4*>(ct + (rb - p * RP + r16) * CP + wn * 16 * NSW + ns * 16 + g4 * 4) = acc[ms][ns];
      }
    }
    lds_barrier();
#pragma unroll
    for (int j = 0; j < RP * TPR / (64 * NWV); ++j) {
      const int idx = tid + 64 * NWV * j, r = idx / TPR, c = idx % TPR * 4;
      const int m = m0 + p * RP + r, n = n0 + c;
      if (p * RP + r < BM && m < M && n < N) store4n(out + (size_t)m * a.ldo + n, *reinterpret_cast<const f32x4*>(ct + r * CP + c), N - n, vec);
    }
    if ((p + 1) * RP < BM) lds_barrier();
  }
}

// ---------------------------------------------------------------------------
template <typename K_>
hipError_t set_lds_attr(K_ kernel) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             160 * 1024);
}

template <typename T, int MS, int NSUB, int NV, bool TL>
hipError_t launch_skinny_l(const SkinnyShape& sh, const GemmArgs& a, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    hipError_t e = set_lds_attr(&gemm_skinny<T, MS, NSUB, NV, TL>);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const dim3 grid(8, sh.m_tiles, (sh.n_tiles * sh.nsplit + 7) / 8);
  hipLaunchKernelGGL((gemm_skinny<T, MS, NSUB, NV, TL>), grid, dim3(64 * WKS), sh.lds, s, a);
  return hipGetLastError();
}
template <typename T, int MS, int NSUB, int NV>
hipError_t launch_skinny_t(const SkinnyShape& sh, const GemmArgs& a, hipStream_t s) {
  return a.wt ? launch_skinny_l<T, MS, NSUB, NV, true>(sh, a, s) : launch_skinny_l<T, MS, NSUB, NV, false>(sh, a, s);
}

template <typename T, int MS, int NSUB>
hipError_t skinny_nv(const SkinnyShape& sh, const GemmArgs& a, hipStream_t s) {
  if constexpr (MS * NSUB <= 4)   // eight steps: within 128 registers for small tiles only
    if (sh.nv == 8) return launch_skinny_t<T, MS, NSUB, 8>(sh, a, s);
  switch (sh.nv) {
    case 2: return launch_skinny_t<T, MS, NSUB, 2>(sh, a, s);
    case 3: return launch_skinny_t<T, MS, NSUB, 3>(sh, a, s);
    case 4: return launch_skinny_t<T, MS, NSUB, 4>(sh, a, s);
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t skinny_t(const SkinnyShape& sh, const GemmArgs& a, hipStream_t s) {
  switch (sh.ms * 10 + sh.nsub) {
    case 11: return skinny_nv<T, 1, 1>(sh, a, s);
    case 12: return skinny_nv<T, 1, 2>(sh, a, s);
    case 21: return skinny_nv<T, 2, 1>(sh, a, s);
    case 22: return skinny_nv<T, 2, 2>(sh, a, s);
    case 41: return skinny_nv<T, 4, 1>(sh, a, s);
    case 42: return skinny_nv<T, 4, 2>(sh, a, s);
    case 24: return skinny_nv<T, 2, 4>(sh, a, s);
    case 44: return skinny_nv<T, 4, 4>(sh, a, s);
  }
  return hipErrorInvalidValue;
}

template <typename T, int MS, int NSUB, int NC>
hipError_t launch_wide_t(const GemmArgs& a, int units, size_t lds, hipStream_t s) {
  static bool attr = false;
  if (!attr) {
    hipError_t e = set_lds_attr(&gemm_wide<T, MS, NSUB, NC>);
    if (e != hipSuccess) return e;
    attr = true;
  }
  hipLaunchKernelGGL((gemm_wide<T, MS, NSUB, NC>), dim3(units), dim3(256), lds, s, a);
  return hipGetLastError();
}

template <typename T, int MS, int NSUB>
hipError_t wide_nc(int nc, const GemmArgs& a, int units, size_t lds, hipStream_t s) {
  switch (nc) {
    case 1: return launch_wide_t<T, MS, NSUB, 1>(a, units, lds, s);
    case 2: return launch_wide_t<T, MS, NSUB, 2>(a, units, lds, s);
    case 4: return launch_wide_t<T, MS, NSUB, 4>(a, units, lds, s);
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t wide_t(const WideShape& sh, const GemmArgs& a, hipStream_t s) {
  switch (sh.ms * 10 + sh.nsub) {
    case 11: return wide_nc<T, 1, 1>(sh.nc, a, sh.units, sh.lds, s);
    case 21: return wide_nc<T, 2, 1>(sh.nc, a, sh.units, sh.lds, s);
    case 41: return wide_nc<T, 4, 1>(sh.nc, a, sh.units, sh.lds, s);
    case 42: return wide_nc<T, 4, 2>(sh.nc, a, sh.units, sh.lds, s);
  }
  return hipErrorInvalidValue;
}


// K % 64 == 0: the direct-to-LDS ring on eight waves (two per SIMD, so one
// wave's LDS and load waits hide behind the other's MFMAs: 12-17% faster than
// four waves on every tile); else the register-staged kernel on four.
template <int MR, int NS>
hipError_t launch_tile_t(const TileShape& sh, const GemmArgs& a, hipStream_t s) {
  if (a.K % 64 == 0) {
    hipLaunchKernelGGL((gemm_tile<MR, NS, 8>), dim3(sh.grid), dim3(512), 0, s, a);
    return hipGetLastError();
  }
  if constexpr (MR % 4 || MR * NS > 64) {   // the ring only
    return hipErrorInvalidValue;
  } else {
    static bool attr = false;
    if (!attr) {
      hipError_t e = set_lds_attr(&gemm_tile_rs<MR / 2, NS>);
      if (e != hipSuccess) return e;
      attr = true;
    }
    const size_t lds = tile_lds_bytes<MR / 2, NS>();
    hipLaunchKernelGGL((gemm_tile_rs<MR / 2, NS>), dim3(sh.grid), dim3(256), lds, s, a);
    return hipGetLastError();
  }
}

// The tiles gemm_tile is instantiated for, as (16-row subtiles, 32-column
// pairs), with the measured time of one 64-wide K-slice of a workgroup on eight
// waves (microseconds, one workgroup per compute unit: bound by the operand
// bytes a compute unit takes in from L2) and the fixed cost of a workgroup
// (pipeline fill, epilogue).
struct TileCand { int mr, ns; double slice_us, fixed_us; };
constexpr int kNumTiles = 8;
constexpr TileCand kTiles[kNumTiles] = {{4, 4, 0.34, 4.0}, {8, 4, 0.47, 5.0}, {16, 4, 0.80, 6.0}, {8, 8, 0.80, 6.0},
                                        {16, 8, 1.6, 8.0},   // from here K % 64 == 0 only
                                        {10, 4, 0.55, 5.3}, {13, 4, 0.67, 5.6}, {13, 8, 1.32, 7.2}};

int cdiv_i(int a, int b) { return (a + b - 1) / b; }

// Time of a skinny launch beyond its fixed latency, in us: the bytes that a
// compute unit takes in at about 48 GB/s, the rounds of its waves, and what
// each split-K partial costs the kernel that sums them.
double skinny_cost(const SkinnyShape& c, int M, int es) {
  const int rows = M - 16 * c.ms * (c.m_tiles - 1) < 16 * c.ms && c.m_tiles == 1 ? M : 16 * c.ms;
  const double per_cu = (double)cdiv_i(c.units, 256);
  const double bytes = (double)(rows + 16 * c.nsub) * c.kper * es;
  const int rounds = cdiv_i(cdiv_i(c.kper, es == 2 ? 32 : 16), WKS * c.nv);
  return per_cu * bytes / 48e3 + 0.5 * (rounds - 1) + 0.08 * (c.nsplit - 1) + 0.05 * c.ms * c.nsub;
}

}  // namespace

int gemm_chunk_k(int et) { return et == ET_BF16 ? 128 : 64; }

// One launch shape of the skinny kernel: 16 ms token rows by 16 nsub W rows
// a workgroup, K in nsplit (a power of two) ranges of whole k-steps.
void skinny_shape(int et, int M, int N, int K, int ms, int nsub, int nsplit, SkinnyShape* sh) {
  const int kstep = gemm_chunk_k(et) / VPL;
  const int sps = cdiv_i(cdiv_i(K, kstep), nsplit);  // steps per split
  sh->ms = ms;
  sh->nsub = nsub;
  sh->n_tiles = cdiv_i(N, 16 * nsub);
  sh->m_tiles = cdiv_i(M, 16 * ms);
  sh->nsplit = nsplit;
  sh->split_log2 = 0;
  while ((1 << sh->split_log2) < nsplit) ++sh->split_log2;
  sh->kper = sps * kstep;
  // the steps spread over the eight waves; eight steps a round (when the
  // registers allow it) before a second round
  const int per_wave = cdiv_i(sps, WKS);
  sh->nv = per_wave <= 2 ? 2 : per_wave == 3 ? 3 : (per_wave == 4 || ms * nsub > 4) ? 4 : 8;
  sh->units = sh->n_tiles * sh->m_tiles * nsplit;
  sh->lds = (size_t)WKS * ms * nsub * 64 * 16;
}

bool skinny_plan(int et, int M, int N, int K, int nsub, bool allow_split, SkinnyShape* sh) {
  const int es = et == ET_BF16 ? 2 : 4, steps = cdiv_i(K, gemm_chunk_k(et) / VPL);
  double best = 1e30;
  for (int ms = 1; ms <= 4; ms *= 2) {
    if (ms > 1 && 16 * (ms / 2) >= M) break;      // half of it covers every row
    for (int ns = nsub; ns <= 4; ns *= 4 / nsub) {
      if (ns == 4 && ms == 1) continue;           // not instantiated
      if (ns == 4 && nsub == 1 && !allow_split) continue;  // EULER and RESID epilogues take one subtile
      for (int sp = 1; sp <= (allow_split ? 8 : 1) && sp <= steps; sp *= 2) {
        if (sp > 1 && (cdiv_i(steps, sp) * (sp - 1)) >= steps) continue;  // an empty last range
        SkinnyShape c;
        skinny_shape(et, M, N, K, ms, ns, sp, &c);
        const double cost = skinny_cost(c, M, es);
        if (cost < best) {
          best = cost;
          *sh = c;
          sh->cost = 2.5 + cost;
        }
      }
      if (nsub == 4) break;
    }
  }
  return best < 1e30;
}

void wide_plan(int et, int M, int N, int K, int nsub, WideShape* sh) {
  const int es = et == ET_BF16 ? 2 : 4;
  const int E = 16 / es;
  const int KC = gemm_chunk_k(et);
  sh->ms = M <= 16 ? 1 : (M <= 32 ? 2 : 4);
  if (nsub == 2) sh->ms = 4;
  sh->nsub = nsub;
  sh->nc = K <= KC ? 1 : (K <= 2 * KC ? 2 : 4);
  const int MT = 16 * sh->ms;
  sh->n_tiles = cdiv_i(N, 64 * nsub);
  sh->m_tiles = cdiv_i(M, MT);
  sh->units = sh->n_tiles * sh->m_tiles;
  sh->lds = (size_t)MT * (sh->nc * KC + E) * es;
}

hipError_t launch_gemm_skinny(int et, const SkinnyShape& sh, GemmArgs a, hipStream_t s) {
  if (sh.units <= 0) return hipSuccess;
  if ((a.wt != 0) != (a.xt != 0)) return hipErrorInvalidValue;   // both operands tiled, or neither
  a.n_tiles = sh.n_tiles;
  a.nsplit = sh.nsplit;
  a.split_log2 = sh.split_log2;
  a.kper = sh.kper;
  return et == ET_BF16 ? skinny_t<bf16_t>(sh, a, s) : skinny_t<float>(sh, a, s);
}

hipError_t launch_gemm_wide(int et, const WideShape& sh, GemmArgs a, hipStream_t s) {
  if (sh.units <= 0) return hipSuccess;
  a.n_tiles = sh.n_tiles;
  a.nsplit = 1;
  return et == ET_BF16 ? wide_t<bf16_t>(sh, a, s) : wide_t<float>(sh, a, s);
}

bool tile_plan(int et, int M, int N, int K, bool allow_split, int force, TileShape* sh) {
  if (et != ET_BF16 || M <= 128 || K % 8 || force >= kNumTiles) return false;
  const int slices = cdiv_i(K, TBK);
  double best = 1e30;
  for (int c = 0; c < kNumTiles; ++c) {
    if (force >= 0 && c != force) continue;
    const TileCand& tc = kTiles[c];
    if (c >= 4 && K % 64) continue;   // the direct-to-LDS ring only
    const int BM = 16 * tc.mr, BN = 32 * tc.ns;
    const int mt = cdiv_i(M, BM), nt = cdiv_i(N, BN);
    const int max_split = (allow_split && force < 0) ? std::min(8, slices) : 1;
    for (int ns = 1; ns <= max_split; ++ns) {
      const int sps = cdiv_i(slices, ns);  // slices per split
      const int nsplit = cdiv_i(slices, sps);
      if (ns > 1 && nsplit != ns) continue;
      const int units = mt * nt * nsplit;
      const double rounds = std::ceil(units / 256.0);
      const double unit_us = tc.fixed_us + sps * tc.slice_us;
      // split partials: written once, read once more by the row kernel
      const double split_us = nsplit > 1 ? 8.0 * M * N * nsplit / 4.0e6 : 0.0;
      const double cost = rounds * unit_us + split_us;
      if (cost < best) {
        best = cost;
        sh->cost = cost;
        sh->mr = tc.mr; sh->ns = tc.ns; sh->nsplit = nsplit; sh->kper = sps * TBK;
        sh->m_tiles = mt; sh->n_tiles = nt; sh->units = units; sh->grid = cdiv_i(units, 8) * 8;
      }
    }
  }
  if (best >= 1e30) return false;
  return true;
}

hipError_t launch_gemm_tile(const TileShape& sh, GemmArgs a, hipStream_t s) {
  if (sh.units <= 0) return hipSuccess;
  a.n_tiles = sh.n_tiles;
  a.m_tiles = sh.m_tiles;
  a.nsplit = sh.nsplit;
  a.kper = sh.kper;
  if ((a.wt || a.xt) && a.K % 64) return hipErrorInvalidValue;   // tiled: the ring kernel's whole slices
  switch (sh.mr * 10 + sh.ns) {
    case 44: return launch_tile_t<4, 4>(sh, a, s);
    case 84: return launch_tile_t<8, 4>(sh, a, s);
    case 164: return launch_tile_t<16, 4>(sh, a, s);
    case 88: return launch_tile_t<8, 8>(sh, a, s);
    case 168: return launch_tile_t<16, 8>(sh, a, s);
    case 104: return launch_tile_t<10, 4>(sh, a, s);
    case 134: return launch_tile_t<13, 4>(sh, a, s);
    case 138: return launch_tile_t<13, 8>(sh, a, s);
  }
  return hipErrorInvalidValue;
}
