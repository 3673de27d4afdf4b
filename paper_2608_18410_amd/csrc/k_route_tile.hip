// Routing scores and selection as two kernels: the token-dependent products on
// matrix cores, split over row blocks, token tiles and slices of the hidden
// size, then one small kernel per 16 tokens that adds the slices and finishes
// the router. Takes every shape, both router kinds and both types; the
// single-kernel and split-K forms (bf16 MLP2, Hr = 128) are faster only for
// many tokens (see route_uses_tiles).
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace rolesub {
namespace {

// ---------------------------------------------------------------------------
// Language pool (Sec. 3.4), as k_route_pool with the language terms as column
// blocks' shares, for either type and router kind and any 16-byte aligned rows:
// block (sample b, 64*VEC columns) means the sample's language rows of its
// columns and forms their share of the language term,
//   pcb[cblk][b][j] = Wl[j, cols] . hbar[b][cols],   Wl = W1[:, d+d_e:] (MLP2)
//                                                     or W_lang (ADDITIVE).
// NJB: 64-row batches of Wl requested
// together (2 for Hr = 128, 1 for the at most 32 rows of W_lang).
constexpr int kLang = 1;
constexpr int kPoolList = 1024;  // tokens listed per pass
template <class T>
struct PoolShared {
  static constexpr int VEC = 16 / sizeof(T);
  int rows[kPoolList];
  int wcnt[4];
  float part[4][64 * VEC];
  float red[4][16][65];
};

template <class T, int NJB>
__device__ __forceinline__ void route_pool_block(const RouteParams& p, PoolShared<T>& sh, int block) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int RU = 16;  // row loads in flight per wave
  const int ncb = (p.d + 64 * VEC - 1) / (64 * VEC);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const bool mlp = p.kind == 0;
  const int nout = mlp ? p.Hr : p.G;
  const int b = block / ncb, cb = block % ncb;
  const uint8_t* ty = p.types + static_cast<size_t>(b) * p.T;
  const int col = cb * 64 * VEC + lane * VEC;
  u32x4 wraw[NJB][16];
  const T* hsample = static_cast<const T*>(p.h) + static_cast<size_t>(b) * p.T * p.d;
  const rsrc_t r_h = make_rsrc(hsample, static_cast<uint32_t>(p.T) * p.d * sizeof(T));
  float acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
  int n_total = 0;
  for (int c0 = 0; c0 < p.T; c0 += kPoolList) {
    const int nc = min(kPoolList, p.T - c0);
    // ascending list of this chunk's language rows (wave ballots + prefix)
    int base = 0;
    for (int s0 = 0; s0 < nc; s0 += 256) {
      const int t = c0 + s0 + tid;
      const bool lang = (s0 + tid < nc) && ty[t] == kLang;
      const uint64_t bal = __ballot(lang);
      const int pre = __popcll(bal & ((1ull << lane) - 1ull));
      if (lane == 0) sh.wcnt[w] = __popcll(bal);
      __syncthreads();
      int woff = base;
      for (int i = 0; i < w; ++i) woff += sh.wcnt[i];
      if (lang) sh.rows[woff + pre] = t;
      base += sh.wcnt[0] + sh.wcnt[1] + sh.wcnt[2] + sh.wcnt[3];
      __syncthreads();
    }
    n_total += base;
    // wave w sums listed rows w, w+4, ...; RU loads in flight per step
    for (int i0 = w; i0 < base; i0 += 4 * RU) {
      u32x4 raw[RU];
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        // the list read at a clamped index: under a branch each of the 16
        // LDS reads is waited for before the next load is issued
        const int i = i0 + 4 * u, t = sh.rows[min(i, base - 1)];
        raw[u] = bload16(r_h, oob_unless(i < base && col < p.d,
                                         static_cast<uint32_t>((static_cast<size_t>(t) * p.d + col) * sizeof(T))));
      }
#pragma unroll
      for (int u = 0; u < RU; ++u) {
        const T* v = reinterpret_cast<const T*>(&raw[u]);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] += tof(v[e]);
      }
    }
    __syncthreads();
  }
  // The language-term weights this block needs, requested after the row
  // loads: loads of a wave complete in issue order, so requested first (128 KB
  // per block at Hr = 128) they held back the token types and language rows
  // behind them.
  const uint32_t Wls = mlp ? 2u * p.d + p.d_e : static_cast<uint32_t>(p.d);
  const rsrc_t r_w = make_rsrc(mlp ? p.W1 : p.W_lang, static_cast<uint32_t>(nout) * Wls * sizeof(T));
  const uint32_t ol = static_cast<uint32_t>((mlp ? p.d + p.d_e : 0) + col) * sizeof(T);
  auto load_w = [&](int j0) {
#pragma unroll
    for (int jb = 0; jb < NJB; ++jb)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int j = j0 + 64 * jb + 16 * w + i;
        wraw[jb][i] = bload16(r_w, oob_unless(j < nout && col < p.d, static_cast<uint32_t>(j) * Wls * sizeof(T) + ol));
      }
  };
  load_w(0);
  // all requested here: the scheduler otherwise moves half of them behind the
  // barrier below, one more round trip
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < VEC; ++e) sh.part[w][lane * VEC + e] = acc[e];
  __syncthreads();
  const float inv = n_total ? 1.f / static_cast<float>(n_total) : 0.f;
  // lane holds pooled columns col..col+VEC-1; wave w takes rows jb+16*w+i
  float hv[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    const int i = lane * VEC + e;
    hv[e] = (((sh.part[0][i] + sh.part[1][i]) + sh.part[2][i]) + sh.part[3][i]) * inv;
  }
  float* dst = p.pcb + (static_cast<size_t>(cb) * p.B + b) * route_ld(nout);
  for (int j0 = 0; j0 < nout; j0 += 64 * NJB) {
    if (j0) load_w(j0);
#pragma unroll
    for (int jh = 0; jh < NJB; ++jh) {
      const int jb = j0 + 64 * jh;
      if (jb >= nout) break;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const T* v = reinterpret_cast<const T*>(&wraw[jh][i]);
        float pd = 0.f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) pd = fmaf(tof(v[e]), hv[e], pd);
        sh.red[w][i][lane] = pd;
      }
      __syncthreads();
      // lane (r = lane/4, q = lane%4) adds lanes 16q..16q+15 of row r, then the
      // four quarters are combined as (q0+q1)+(q2+q3)
      const int r = lane >> 2, q = lane & 3;
      float sum = 0.f;
#pragma unroll
      for (int k = 0; k < 16; ++k) sum += sh.red[w][r][16 * q + k];
      sum += __shfl_xor(sum, 1);
      sum += __shfl_xor(sum, 2);
      const int j = jb + 16 * w + r;
      if (q == 0 && j < nout) dst[j] = sum;
      __syncthreads();
    }
  }
}

// The folded role term of row j and role c (zero unless ok): W1[j, d : d+d_e] .
// E[c], or alpha_role W_role[j][c]. VECT: d, d_e multiples of 16 bytes, rows
// 16-byte aligned.
template <class T, bool VECT>
__device__ __forceinline__ float role_term(const RouteParams& p, int j, int c, bool ok) {
  constexpr int VEC = 16 / sizeof(T);
  if (p.kind != 0) return ok ? p.alpha_role * tof(static_cast<const T*>(p.W_role)[j * p.C + c]) : 0.f;
  const uint32_t W1s = 2u * p.d + p.d_e;
  float acc = 0.f;
  if constexpr (VECT) {
    const rsrc_t r_w = make_rsrc(p.W1, static_cast<uint32_t>(p.Hr) * W1s * sizeof(T));
    const rsrc_t r_e = make_rsrc(p.E, static_cast<uint32_t>(p.C * p.d_e) * sizeof(T));
    const uint32_t ow = (static_cast<uint32_t>(j) * W1s + p.d) * sizeof(T);
    const uint32_t oe = static_cast<uint32_t>(c * p.d_e) * sizeof(T);
    // 16 loads of each operand in flight: one round trip for d_e <= 16*VEC
    for (int m0 = 0; m0 < p.d_e; m0 += 16 * VEC) {
      u32x4 wv[16], ev[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const bool in = ok && m0 + u * VEC < p.d_e;
        const uint32_t m = static_cast<uint32_t>(m0 + u * VEC) * sizeof(T);
        wv[u] = bload16(r_w, oob_unless(in, ow + m));
        ev[u] = bload16(r_e, oob_unless(in, oe + m));
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const T* a = reinterpret_cast<const T*>(&wv[u]);
        const T* x = reinterpret_cast<const T*>(&ev[u]);
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc = fmaf(tof(a[i]), tof(x[i]), acc);
      }
    }
  } else if (ok) {
    const T* a = static_cast<const T*>(p.W1) + static_cast<size_t>(j) * W1s + p.d;
    const T* x = static_cast<const T*>(p.E) + static_cast<size_t>(c) * p.d_e;
    for (int m = 0; m < p.d_e; ++m) acc = fmaf(tof(a[m]), tof(x[m]), acc);
  }
  return acc;
}

// The pool for the one-kernel forms where d is no multiple of 512 (k_route_pool
// takes the others); blocks past the samples' fold F[Hr][C], as there.
__global__ __launch_bounds__(256) void k_route_pool_any(RouteParams p) {
  __shared__ PoolShared<bf16> sh;
  const int nb = p.B * ((p.d + 511) / 512);
  if (static_cast<int>(blockIdx.x) < nb) {
    route_pool_block<bf16, 2>(p, sh, blockIdx.x);
    return;
  }
  const int fb = blockIdx.x - nb, e = fb * 256 + threadIdx.x, j = e / p.C;
  const float f = role_term<bf16, true>(p, j, e - j * p.C, j < p.Hr);
  if (j < p.Hr) p.F[e] = f;
  if (p.rcnt) {
    const int ntiles = static_cast<int>((static_cast<size_t>(p.B) * p.T + kRouteSkTok - 1) / kRouteSkTok);
    const int nfb = (p.Hr * p.C + 255) / 256;
    for (int i = e; i < ntiles; i += nfb * 256) p.rcnt[i] = 0;
  }
}

// ---------------------------------------------------------------------------
// Products. The rows are the 16-row blocks of W_main (W1_h or W_tok, nbm
// blocks) followed by those of W_r; a workgroup computes NRB of them for 64
// tokens over one slice of the hidden size and stores the accumulators as
// they stand: part[slice][tile][block][wave] holds the 16 x 16 products of the
// tile's tokens 16*wave.. as one f32x4 per lane (token l16, rows 4*g4 ..).
//
// Both operands stream through a ring of LDS stages of 128 bytes per row (64
// bf16 or 32 f32 columns), filled by asynchronous LDS DMA issued several
// stages ahead; rows are stored with their 16-byte pieces XOR-swizzled, which makes
// the fragment reads of 16 rows free of bank conflicts. A 16-byte piece per
// lane is one operand of a bf16 16x16x32 MFMA, or of four f32 16x16x4 MFMAs
// (element i of each lane; the k order is the same on both sides).
//
// What bounds it: with few tokens the chain of a stage (wait, barrier, fragment
// reads, 6 MFMAs: about 400 ns), so a workgroup takes three row blocks (two for
// the additive router's) and the rows, tokens and slices are spread over
// workgroups; where all of them get a CU to themselves (DEEP) a step covers two
// stages (one prefix, both kernels: 21.6 against 23.2 us). With many tokens the
// hidden states' stream. The language pool runs beside the products in the same
// launch. Measured, both kernels, against the forms they replace (d = 4096, 48
// language tokens of 177): bf16 additive router, 64 prefixes, 31 us (93 MB of
// hidden states) against 1270 of one workgroup per token; bf16 MLP2, one
// prefix, 21.6 us against 31.8 of the split-K form's workgroups; f32 MLP2, two
// prefixes, 23 against 162.
constexpr int kTok = 64;

struct TileParams {
  float* part;
  float *Ff, *W2f, *brf, *bf;  // folded operands (route_fold_floats)
  int S, MB, nbm, RC;   // slices, row blocks in all and of W_main, row chunks of NRB blocks
  int npool, nfold;     // language-pool and folding blocks at the front of the grid
  int ncb;              // shares of the language term to add (0: cb holds it)
  int ntile;            // tiles of this launch
  size_t tok0;          // first token of this launch
};

__device__ __forceinline__ int swz8(int r) { return (r >> 1) & 7; }

template <class T>
__device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c);
template <>
__device__ __forceinline__ f32x4 mma<bf16>(u32x4 a, u32x4 b, f32x4 c) {
  return mfma_16x16x32(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c);
}
template <>
__device__ __forceinline__ f32x4 mma<float>(u32x4 a, u32x4 b, f32x4 c) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i]), __uint_as_float(b[i]), c, 0, 0, 0);
  return c;
}

// The finishing kernel's operands, one thread per float:
//   Ff[m][cb][lane][k] = F[16 m + lane % 16][16 cb + 4 k + lane / 16], zero past
//                        the rows and roles;
//   W2f[m][q][s][i]    = W2[s][16 m + 4 q + i], zero past Hr;
//   brf                  role biases, -inf past C;
//   bf                   biases of the main rows (b1; alpha_lang b_lang + b_tok).
template <class T, bool VECT>
__device__ __forceinline__ void fold_block(const RouteParams& p, const TileParams& t, int e) {
  const int RB = t.MB - t.nbm, nmain = p.kind == 0 ? p.Hr : p.G;
  const int nF = t.nbm * RB * 256, nW = p.kind == 0 ? t.nbm * p.G * 16 : 0;
  if (e < nF) {
    const int lane = (e >> 2) & 63, cb = (e >> 8) % RB, m = (e >> 8) / RB;
    const int j = 16 * m + (lane & 15), c = 16 * cb + 4 * (e & 3) + (lane >> 4);
    t.Ff[e] = role_term<T, VECT>(p, j, c, j < nmain && c < p.C);
    return;
  }
  e -= nF;
  if (e < nW) {
    const int s = (e >> 2) % p.G, mq = (e >> 2) / p.G, j = 4 * mq + (e & 3);
    t.W2f[e] = j < p.Hr ? tof(static_cast<const T*>(p.W2)[static_cast<size_t>(s) * p.Hr + j]) : 0.f;
    return;
  }
  e -= nW;
  if (e < 16 * RB) {
    t.brf[e] = e < p.C ? tof(static_cast<const T*>(p.b_r)[e]) : -INFINITY;
    return;
  }
  e -= 16 * RB;
  if (e < 16 * t.nbm) {
    float v = 0.f;
    if (e < nmain)
      v = p.kind == 0 ? tof(static_cast<const T*>(p.b1)[e])
                      : fmaf(p.alpha_lang, tof(static_cast<const T*>(p.b_lang)[e]), tof(static_cast<const T*>(p.b_tok)[e]));
    t.bf[e] = v;
  }
}

template <class T>
__global__ __launch_bounds__(256) void k_route_fold(RouteParams p, TileParams t) {
  fold_block<T, false>(p, t, blockIdx.x * 256 + threadIdx.x);
}

// DMA: rows and row strides are multiples of 16 bytes, 16-byte aligned.
// Otherwise the stages are filled through registers.
template <class T, int NRB, bool DMA, bool DEEP>
__global__ __launch_bounds__(256) void k_route_tile(RouteParams p, TileParams t) {
  constexpr int STEP = DEEP ? 2 : 1;  // stages per barrier
  constexpr int NB = !DMA ? 2 : DEEP ? 10 : NRB == 2 ? 4 : 5;
  constexpr int kWB = NRB * 16 * 128, kStage = kWB + kTok * 128;
  constexpr int NL = 2 * NRB + kTok / 8;  // 1 KB wave-loads per stage
  constexpr int UMAX = (NL + 3) / 4, UMIN = NL / 4;
  constexpr int EPC = 128 / sizeof(T);    // columns per stage
  constexpr size_t kShm = DMA && sizeof(PoolShared<T>) > NB * kStage ? sizeof(PoolShared<T>) : NB * kStage;
  __shared__ __attribute__((aligned(16))) char ring[kShm];
  if constexpr (DMA) {
    if (static_cast<int>(blockIdx.x) < t.npool) {
      route_pool_block<T, NRB == 3 ? 2 : 1>(p, *reinterpret_cast<PoolShared<T>*>(ring), blockIdx.x);
      return;
    }
    if (static_cast<int>(blockIdx.x) < t.npool + t.nfold) {
      fold_block<T, true>(p, t, (blockIdx.x - t.npool) * 256 + threadIdx.x);
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // slices and row chunks fastest: consecutive workgroups (on different XCDs)
  // read the same tile's hidden states
  const int lin = blockIdx.x - t.npool - t.nfold;
  const int s = lin % t.S, rest = lin / t.S, rc = rest % t.RC, tile = rest / t.RC;
  const int d = p.d, C = p.C;
  const bool mlp = p.kind == 0;
  const int nmain = mlp ? p.Hr : p.G;
  const uint32_t Ws = (mlp ? 2u * d + p.d_e : static_cast<uint32_t>(d)) * sizeof(T);  // row bytes of W_main
  const uint32_t dB = static_cast<uint32_t>(d) * sizeof(T);
  const size_t N = static_cast<size_t>(p.B) * p.T, tok0 = t.tok0 + static_cast<size_t>(tile) * kTok;
  const int nvalid = static_cast<int>(N - tok0 < kTok ? N - tok0 : kTok);
  const char* hbase = static_cast<const char*>(p.h) + tok0 * dB;
  const void* wmain = mlp ? p.W1 : p.W_tok;
  const int nch = (d + EPC - 1) / EPC;
  const int c0 = static_cast<int>(static_cast<int64_t>(s) * nch / t.S);
  const int c1 = static_cast<int>(static_cast<int64_t>(s + 1) * nch / t.S);
  const int r0 = rc * NRB * 16;  // first row, in the numbering of part

  f32x4 acc[NRB];
#pragma unroll
  for (int m = 0; m < NRB; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int th = 16 * w + l16;

  const rsrc_t r_h = make_rsrc(hbase, static_cast<uint32_t>(nvalid) * dB);
  const rsrc_t r_w = make_rsrc(wmain, static_cast<uint32_t>(nmain) * Ws);
  const rsrc_t r_r = make_rsrc(p.W_r, static_cast<uint32_t>(C) * dB);
  // Wave-load j = w + 4u < NL of a stage: row groups 8j.. for j < 2 NRB
  // (both halves of a block, so one matrix each), then token rows. Lane i
  // carries row 8j + i/8, LDS piece i%8, global piece (i%8) ^ swizzle.
  const int ri = lane >> 3, piece = lane & 7;
  uint32_t base_off[UMAX], pcol[UMAX];
#pragma unroll
  for (int u = 0; u < UMAX; ++u) {
    const int j = w + 4 * u;
    uint32_t off = kOOB;
    int r = 8 * j + ri;
    if (j < 2 * NRB) {
      const int gr = r0 + r, rr = gr - 16 * t.nbm;
      if (rr < 0) {
        if (gr < nmain) off = static_cast<uint32_t>(gr) * Ws;
      } else if (rr < C) {
        off = static_cast<uint32_t>(rr) * dB;
      }
    } else {
      r = 8 * (j - 2 * NRB) + ri;
      if (r < nvalid) off = static_cast<uint32_t>(r) * dB;
    }
    base_off[u] = off;
    pcol[u] = 16u * (piece ^ swz8(r));
  }

  if constexpr (DMA) {
    const uint32_t ring_base = lds_addr(ring);
    auto issue_one = [&](int i, int u) {
      const int j = w + 4 * u;
      if (u >= UMIN && j >= NL) return;  // the last load of the waves that have one fewer
      const uint32_t col = static_cast<uint32_t>(c0 + i) * 128u + pcol[u];
      // stages past the slice and columns past d load as zeros
      const bool ok = (c0 + i < c1) & (col < dB) & (base_off[u] != kOOB);
      const uint32_t off = oob_unless(ok, base_off[u] + col);
      const uint32_t dst = ring_base + (i % NB) * kStage + 1024u * j;
      if (j >= 2 * NRB) dma16(r_h, off, dst);
      else if (r0 + 8 * j < 16 * t.nbm) dma16(r_w, off, dst);
      else dma16(r_r, off, dst);
    };
#pragma unroll
    for (int i = 0; i < NB - STEP; ++i)
#pragma unroll
      for (int u = 0; u < UMAX; ++u) issue_one(i, u);
    // (stages past the slice are zeros: an odd slice's last step adds nothing)
    for (int i = 0; i < c1 - c0; i += STEP) {
      // stages i .. have landed once at most NB - 2 STEP younger ones are pending
      if (UMAX == UMIN || w < NL % 4) wait_vmcnt<UMAX * (NB - 2 * STEP)>();
      else wait_vmcnt<UMIN * (NB - 2 * STEP)>();
      __syncthreads();
      u32x4 hb[2 * STEP], af[2 * STEP][NRB];
#pragma unroll
      for (int ks = 0; ks < 2 * STEP; ++ks) {
        const char* st = ring + ((i + ks / 2) % NB) * kStage;
        const int piece16 = 4 * (ks & 1) + g4;
        hb[ks] = *reinterpret_cast<const u32x4*>(st + kWB + th * 128 + 16 * (piece16 ^ swz8(th)));
#pragma unroll
        for (int m = 0; m < NRB; ++m) {
          const int r = 16 * m + l16;
          af[ks][m] = *reinterpret_cast<const u32x4*>(st + r * 128 + 16 * (piece16 ^ swz8(r)));
        }
      }
      // the refill of the stages released at this barrier between the MFMAs
      constexpr int NM = 2 * NRB * STEP, NU = UMAX * STEP;
#pragma unroll
      for (int q = 0; q < NM; ++q) {
        acc[q % NRB] = mma<T>(af[q / NRB][q % NRB], hb[q / NRB], acc[q % NRB]);
#pragma unroll
        for (int u = 0; u < NU; ++u)
          if (u * NM / NU == q) issue_one(i + NB - STEP + u / UMAX, u % UMAX);
      }
    }
    wait_vmcnt<0>();  // trailing dummy loads land before the LDS is released
  } else {
    // 16 bytes a lane through registers, two stages ahead of their use; the piece
    // that a row ends in element by element. Bound by the round trip of a stage's
    // loads. Measured, whole calls at d = 1001, Hr = 128: 8 tokens 29 us, 16 x 177
    // 46, against 61 and 92 with every element loaded by itself for the stage at
    // hand, and 47 and 204 with one workgroup per token.
    struct Stage {
      u32x4 v[UMAX];
    };
    const bool tail = d % (16 / static_cast<int>(sizeof(T))) != 0;
    auto load = [&](Stage& x, int c) {
#pragma unroll
      for (int u = 0; u < UMAX; ++u) {
        const int j = w + 4 * u;
        if (u >= UMIN && j >= NL) break;  // the last load of the waves that have one fewer
        const uint32_t col = static_cast<uint32_t>(c) * 128u + pcol[u];
        const uint32_t off = oob_unless((c < c1) & (col + 16u <= dB) & (base_off[u] != kOOB), base_off[u] + col);
        const rsrc_t r = j >= 2 * NRB ? r_h : r0 + 8 * j < 16 * t.nbm ? r_w : r_r;
        x.v[u] = bload16(r, off);
        if (tail && c == nch - 1 && c < c1 && col < dB && col + 16u > dB && base_off[u] != kOOB) {
          const char* src = (j >= 2 * NRB ? hbase : static_cast<const char*>(r0 + 8 * j < 16 * t.nbm ? wmain : p.W_r)) +
                            base_off[u] + col;
          T e[16 / sizeof(T)];
#pragma unroll
          for (uint32_t i = 0; i < 16 / sizeof(T); ++i)
            e[i] = col + i * sizeof(T) < dB ? reinterpret_cast<const T*>(src)[i] : fromf<T>(0.f);
          __builtin_memcpy(&x.v[u], e, 16);
        }
      }
    };
    auto step = [&](Stage& x, int c) {
      char* st = ring + ((c - c0) & 1) * kStage;
#pragma unroll
      for (int u = 0; u < UMAX; ++u) {
        const int j = w + 4 * u;
        if (u >= UMIN && j >= NL) break;
        *reinterpret_cast<u32x4*>(st + 1024 * j + 16 * lane) = x.v[u];
      }
      load(x, c + 2);
      __syncthreads();  // (two stages: the next step writes the other one)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const u32x4 hb = *reinterpret_cast<const u32x4*>(st + kWB + th * 128 + 16 * ((4 * ks + g4) ^ swz8(th)));
#pragma unroll
        for (int m = 0; m < NRB; ++m) {
          const int r = 16 * m + l16;
          acc[m] = mma<T>(*reinterpret_cast<const u32x4*>(st + r * 128 + 16 * ((4 * ks + g4) ^ swz8(r))), hb, acc[m]);
        }
      }
    };
    Stage xa, xb;
    load(xa, c0);
    load(xb, c0 + 1);
    for (int c = c0; c < c1; c += 2) {
      step(xa, c);
      if (c + 1 < c1) step(xb, c + 1);
    }
  }
  f32x4* out = reinterpret_cast<f32x4*>(t.part) +
               ((static_cast<size_t>(s) * t.ntile + tile) * t.MB + rc * NRB) * 256 + tid;
#pragma unroll
  for (int m = 0; m < NRB; ++m)
    if (rc * NRB + m < t.MB) out[m * 256] = acc[m];
}

// ---------------------------------------------------------------------------
// Finish: one workgroup of eight waves per 16 tokens. Wave w owns the main row
// blocks m = w, w + 8, ...; lane (token l16, quarter g4) holds rows 16m + 4g4 +
// i, the layout of the products. Where the one-kernel forms take a call of more
// tokens (route_uses_tiles), every sum runs in their order, so that both give the
// same bits: the halves of the hidden size; the column blocks' shares of the
// language term, then the bias; F a on the f32 matrix cores; W2 per row block,
// then over the blocks, then over the lane quarters. The ranking gives every
// (token, group) a thread. With one or two waves per SIMD it is bound by the
// instructions of one wave, so every operand is a 16-byte load at one lane
// offset plus a scalar one (F, W2 and the biases folded into that layout by the
// first kernel); with masked element loads and 64-bit addresses it ran 10-18 us.
constexpr int kFinW = 8;

__device__ __forceinline__ f32x4 loadf4(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, static_cast<int>(voff), static_cast<int>(soff), 0));
}

// KIND as in RouteParams; GP >= G bounds the group loops (8, 16, 32); CB >= RB
// the role blocks' (1 or 4)
template <class T, int KIND, int GP, int CB>
__global__ __launch_bounds__(64 * kFinW) void k_route_finish(RouteParams p, TileParams t) {
  constexpr int SL = sizeof(T) == 2 ? kRouteSlicesBf16 : kRouteSlicesF32;  // slices at most, requested together
  constexpr int NB = KIND == 0 ? kFinW : (GP + 15) / 16;  // waves with row blocks
  constexpr int GC = GP < 8 ? GP : 8;                     // groups of W2 held at a time
  __shared__ float gsum[KIND == 0 ? kFinW : 1][KIND == 0 ? GP : 1][KIND == 0 ? 65 : 1];
  __shared__ __attribute__((aligned(16))) f32x4 rsum[CB][kFinW][64];
  __shared__ __attribute__((aligned(16))) float as[kFinW][16][16 * CB + 4];  // role weights per wave
  __shared__ float sc[16][33];
  __shared__ __attribute__((aligned(16))) uint32_t keys[16][36];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = p.G, nmain = KIND == 0 ? p.Hr : G, S = t.S;
  const size_t N = static_cast<size_t>(p.B) * p.T;
  const size_t t16 = t.tok0 + static_cast<size_t>(blockIdx.x) * 16;
  const int nv = static_cast<int>(N - t16 < 16 ? N - t16 : 16);
  const int RB = t.MB - t.nbm;
  // this tile quarter's products: slice s of block m at s * sstep + 4096 m
  const uint32_t sstep = static_cast<uint32_t>(t.ntile) * t.MB * 4096u;
  const uint32_t tbase = ((blockIdx.x >> 2) * t.MB * 4u + (blockIdx.x & 3)) * 1024u;
  const rsrc_t r_part = make_rsrc(t.part, clamp_bytes(static_cast<size_t>(S) * sstep));
  const uint32_t lo = 16u * lane;
  // language terms of the (at most 16) samples the tokens belong to: share u
  // starts at lterm + u * B * ld
  const int b0 = __builtin_amdgcn_readfirstlane(static_cast<int>(t16 / p.T));
  const uint32_t tin = static_cast<uint32_t>(t16 - static_cast<size_t>(b0) * p.T) + min(l16, nv - 1);
  const uint32_t db = tin / static_cast<uint32_t>(p.T);
  const int ld = static_cast<int>(route_ld(nmain));
  const float* lterm = (t.ncb ? p.pcb : p.cb) + static_cast<size_t>(b0) * ld;
  const int ns = t.ncb ? t.ncb : 1;
  const size_t lstep = static_cast<size_t>(p.B) * ld;
  const uint32_t lbytes = static_cast<uint32_t>(min(16, p.B - b0)) * ld * 4u;
  const rsrc_t r_F = make_rsrc(t.Ff, static_cast<uint32_t>(t.nbm) * RB * 1024u);
  const rsrc_t r_W = make_rsrc(t.W2f, KIND == 0 ? static_cast<uint32_t>(t.nbm) * G * 64u : 0u);

  // A row block's operands: its first SL slices, the first 8 shares of the
  // language term, its bias and fragment of F, and W2 of the first GC groups
  struct Block {
    f32x4 v[SL], lt[8], bias, f, w2[KIND == 0 ? GC : 1];
  };
  auto lt_row = [&](int u, int m) {
    const rsrc_t r = make_rsrc(lterm + static_cast<size_t>(min(u, ns - 1)) * lstep, lbytes);
    // rows past ld (only in the last block) are not used
    return __builtin_bit_cast(f32x4, bload16(r, (db * ld + 16u * m + 4u * g4) * 4u));
  };
  auto w2_row = [&](int m, int s) { return loadf4(r_W, 16u * G * g4, 64u * G * m + 16u * s); };  // past G: unused or zero
  auto load = [&](Block& x, int m) {
#pragma unroll
    for (int u = 0; u < SL; ++u) x.v[u] = loadf4(r_part, lo, tbase + 4096u * m + min(u, S - 1) * sstep);
#pragma unroll
    for (int u = 0; u < 8; ++u) x.lt[u] = lt_row(u, m);
    x.bias = reinterpret_cast<const f32x4*>(t.bf)[4 * m + g4];
    x.f = loadf4(r_F, lo, 1024u * RB * m);
    if constexpr (KIND == 0) {
#pragma unroll
      for (int s = 0; s < GC; ++s) x.w2[s] = w2_row(m, s);
    }
  };

  // ---- requested together: the wave's first main block, its share of the
  // role blocks' slices (slice w), and what the end needs
  Block x;
  const bool mine = w < NB && w < t.nbm;
  const f32x4* brf = reinterpret_cast<const f32x4*>(t.brf);
  const f32x4 rb = brf[g4];
  f32x4 rv = loadf4(r_part, lo, tbase + 4096u * t.nbm + min(w, S - 1) * sstep);
  if (mine) load(x, w);
  const int tt = tid >> 5, ts = tid & 31;  // the selection's token and group
  const int type = p.mask ? p.types[t16 + min(tt, nv - 1)] : 0;
  const float b2v = KIND == 0 ? tof(static_cast<const T*>(p.b2)[min(ts, G - 1)]) : 0.f;
  static_assert(SL <= kFinW, "a wave per slice of the role blocks");
  for (int cb = 0; cb < RB; ++cb) {
    if (cb) rv = loadf4(r_part, lo, tbase + 4096u * (t.nbm + cb) + min(w, S - 1) * sstep);
    rsum[cb][w][lane] = rv;
  }
  __syncthreads();

  const int half = (S + 1) >> 1;
  if (mine) {
    // ---- role weights a (Eq. latentrole), role 16cb + 4g4 + i of token l16
    f32x4 a[CB];
    float mx = -INFINITY, sm = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      if (cb < RB) {
        f32x4 y0 = rsum[cb][0][lane], y1 = {0.f, 0.f, 0.f, 0.f};
        for (int v = 1; v < half; ++v) y0 += rsum[cb][v][lane];
        for (int v = half; v < S; ++v) y1 += rsum[cb][v][lane];
        a[cb] = (y0 + y1) + (cb ? brf[4 * cb + g4] : rb);  // -inf past C
#pragma unroll
        for (int i = 0; i < 4; ++i) mx = fmaxf(mx, a[cb][i]);
      }
    }
    mx = max_xor32(max_xor16(mx));
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      if (cb < RB)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float e = expf(a[cb][i] - mx);
          a[cb][i] = 16 * cb + 4 * g4 + i < p.C ? e : 0.f;
          sm += a[cb][i];
        }
    sm = add_xor32(add_xor16(sm));
    const float isum = 1.f / sm;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
      if (cb < RB) *reinterpret_cast<f32x4*>(&as[w][l16][16 * cb + 4 * g4]) = a[cb] * isum;
    // (read back by this wave only: the k order of F a is role 4k + g4)
    if (p.priority && w == 0 && g4 == 0 && l16 < nv) {
      float pr = 0.f;
      for (int c = 0; c < p.C; ++c) pr = fmaf(tof(static_cast<const T*>(p.w_pri)[c]), as[0][l16][c], pr);
      p.priority[t16 + l16] = pr;
    }

    float gam[KIND == 0 ? GP : 1];
    for (int m = w; m < t.nbm; m += NB) {
      if (m != w) load(x, m);
      const int j0 = 16 * m + 4 * g4;  // this lane's rows j0 .. j0 + 3
      // the slices of either half in order, then the halves
      f32x4 y = x.v[0], y1 = {0.f, 0.f, 0.f, 0.f}, lt = x.lt[0];
#pragma unroll
      for (int u = 1; u < SL; ++u) {
        if (u < half) y += x.v[u];
        else if (u < S) y1 += x.v[u];
      }
      y += y1;
      // F a: row l16 of the block, role 16cb + 4k + g4
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        if (cb < RB) {
          const f32x4 f = cb ? loadf4(r_F, lo, 1024u * (RB * m + cb)) : x.f;
#pragma unroll
          for (int k = 0; k < 4; ++k)
            y = __builtin_amdgcn_mfma_f32_16x16x4f32(f[k], as[w][l16][16 * cb + 4 * k + g4], y, 0, 0, 0);
        }
      // the column blocks' shares in order, then the bias
#pragma unroll
      for (int u = 1; u < 8; ++u)
        if (u < ns) lt += x.lt[u];
      for (int u = 8; u < ns; u += 8) {
        f32x4 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = lt_row(u + e, m);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (u + e < ns) lt += v[e];
      }
      if (t.ncb) lt = KIND == 0 ? lt + x.bias : lt * p.alpha_lang + x.bias;
      y += lt;
      if constexpr (KIND == 0) {
        float g[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) g[i] = j0 + i < nmain ? gelu_exact(y[i]) : 0.f;
#pragma unroll
        for (int s = 0; s < GP; ++s) {
          if (s >= GC && s % GC == 0) {
#pragma unroll
            for (int e = 0; e < GC; ++e) x.w2[e] = w2_row(m, s + e);
          }
          const f32x4 w2 = x.w2[s % GC];
          float v = w2[0] * g[0];
          v = fmaf(w2[1], g[1], v);
          v = fmaf(w2[2], g[2], v);
          v = fmaf(w2[3], g[3], v);
          gam[s] = m == w ? v : gam[s] + v;
        }
      } else {
        // the block is the score block itself
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[l16][j0 + i] = y[i];
      }
    }
    if constexpr (KIND == 0) {
#pragma unroll
      for (int s = 0; s < GP; ++s) gsum[w][s][lane] = gam[s];
    }
  }
  __syncthreads();
  // ---- selection: thread (token tt, group s); the 32 lanes of a token hold
  // its groups, so counts and masks are ballots
  const int s = ts;
  const size_t tok = t16 + tt;
  const bool live = tt < nv && s < G;
  float g;
  if constexpr (KIND == 0) {
    // over the row blocks, then over the lane quarters
    const int sg = min(s, GP - 1);
    f32x4 q;
#pragma unroll
    for (int e = 0; e < 4; ++e) q[e] = gsum[0][sg][16 * e + tt];
    for (int v = 1; v < min(kFinW, t.nbm); ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) q[e] += gsum[v][sg][16 * e + tt];
    g = ((q[0] + q[1]) + (q[2] + q[3])) + b2v;
  } else {
    g = sc[tt][min(s, 16 * NB - 1)];
  }
  if (live && p.scores_out) p.scores_out[tok * G + s] = g;
  if (!p.mask) return;
  const uint32_t key = live ? order_key(g) : 0u;
  keys[tt][s] = key;  // read by this wave only
  const int sh = lane & 32;
  const int n_above = __popc(static_cast<uint32_t>(__ballot(live && g > p.tau) >> sh));
  const int K = budget_k(p.mode, p.k_by_type, type, p.tau, p.kmin, p.kmax, G, n_above);
  int rank = 0;
#pragma unroll
  for (int u0 = 0; u0 < GP; u0 += 4) {
    if (u0 >= G) break;
    const u32x4 ku = *reinterpret_cast<const u32x4*>(&keys[tt][u0]);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      rank += static_cast<int>((u0 + e < G) & ((ku[e] > key) | ((ku[e] == key) & (u0 + e < s))));
  }
  const bool kept = live && rank < K;
  const uint32_t m = static_cast<uint32_t>(__ballot(kept) >> sh);
  if (!live) return;
  const int nk = __popc(m);
  if (s == 0) {
    p.mask[tok] = m;
    if (p.count) p.count[tok] = static_cast<uint8_t>(nk);
  }
  if (p.idx) {
    const int below = __popc(m & ((1u << s) - 1u));
    p.idx[tok * G + (kept ? below : nk + (s - below))] = kept ? static_cast<uint8_t>(s) : 0xFF;
  }
}

struct Plan {
  int MB, nbm, NRB, RC, S;
  size_t tiles;
};

Plan make_plan(const RouteParams& p, bool bf16) {
  Plan q;
  q.nbm = route_tile_blocks(p.Hr, p.G, 0, p.kind);
  q.MB = route_tile_blocks(p.Hr, p.G, p.C, p.kind);
  q.NRB = route_tile_rows(q.MB);
  q.RC = (q.MB + q.NRB - 1) / q.NRB;
  q.tiles = (static_cast<size_t>(p.B) * p.T + kTok - 1) / kTok;
  q.S = route_tile_slices(p.d, q.MB, p.kind, bf16);
  return q;
}

template <class T, bool DMA>
void launch_products(const Plan& q, const RouteParams& p, const TileParams& t, unsigned grid, hipStream_t s) {
  const dim3 g(grid), blk(256);
  // one workgroup per CU anyway: long ring, two stages per barrier (bf16; an f32
  // stage is a microsecond of matrix-core time)
  constexpr bool kDeep = DMA && sizeof(T) == 2;
  if (kDeep && grid <= 256) {
    if (q.NRB == 2) hipLaunchKernelGGL((k_route_tile<T, 2, DMA, kDeep>), g, blk, 0, s, p, t);
    else hipLaunchKernelGGL((k_route_tile<T, 3, DMA, kDeep>), g, blk, 0, s, p, t);
  } else {
    if (q.NRB == 2) hipLaunchKernelGGL((k_route_tile<T, 2, DMA, false>), g, blk, 0, s, p, t);
    else hipLaunchKernelGGL((k_route_tile<T, 3, DMA, false>), g, blk, 0, s, p, t);
  }
}

template <class T, int KIND, int GP>
void launch_finish_g(const RouteParams& p, const TileParams& t, unsigned grid, hipStream_t s) {
  const dim3 blk(64 * kFinW);
  if (p.C <= 16) hipLaunchKernelGGL((k_route_finish<T, KIND, GP, 1>), dim3(grid), blk, 0, s, p, t);
  else hipLaunchKernelGGL((k_route_finish<T, KIND, GP, 4>), dim3(grid), blk, 0, s, p, t);
}

template <class T>
void launch_finish(const RouteParams& p, const TileParams& t, unsigned grid, hipStream_t s) {
  if (p.kind == 0) {
    if (p.G <= 8) launch_finish_g<T, 0, 8>(p, t, grid, s);
    else if (p.G <= 16) launch_finish_g<T, 0, 16>(p, t, grid, s);
    else launch_finish_g<T, 0, 32>(p, t, grid, s);
  } else {
    if (p.G <= 16) launch_finish_g<T, 1, 16>(p, t, grid, s);
    else launch_finish_g<T, 1, 32>(p, t, grid, s);
  }
}

template <class T>
hipError_t launch_tile_t(const RouteParams& p, const Plan& q, size_t part_bytes, hipStream_t s) {
  constexpr int VEC = 16 / sizeof(T);
  const size_t N = static_cast<size_t>(p.B) * p.T;
  const uintptr_t bases = reinterpret_cast<uintptr_t>(p.h) | reinterpret_cast<uintptr_t>(p.W_r) |
                          (p.kind == 0 ? reinterpret_cast<uintptr_t>(p.W1) | reinterpret_cast<uintptr_t>(p.E)
                                       : reinterpret_cast<uintptr_t>(p.W_tok) | reinterpret_cast<uintptr_t>(p.W_lang));
  const bool dma = (bases & 15) == 0 && p.d % VEC == 0 && (p.kind != 0 || p.d_e % VEC == 0);
  TileParams t = {};
  t.Ff = p.part;
  t.W2f = t.Ff + static_cast<size_t>(q.nbm) * (q.MB - q.nbm) * 256;
  t.brf = t.W2f + (p.kind == 0 ? static_cast<size_t>(q.nbm) * p.G * 16 : 0);
  t.bf = t.brf + static_cast<size_t>(q.MB - q.nbm) * 16;
  const size_t fold = route_fold_floats(p.Hr, p.G, p.C, p.kind);
  t.part = p.part + fold;
  part_bytes -= fold * sizeof(float);
  t.S = q.S;
  t.MB = q.MB;
  t.nbm = q.nbm;
  t.RC = q.RC;
  const int ncb = (p.d + 64 * VEC - 1) / (64 * VEC);
  const unsigned nfold = static_cast<unsigned>((fold + 255) / 256);  // a thread per float
  if (dma) {
    t.ncb = ncb;
  } else {
    launch_pool_proj(p, sizeof(T) == 2, s);
    hipLaunchKernelGGL(k_route_fold<T>, dim3(nfold), dim3(256), 0, s, p, t);
  }
  static_assert(16 * kTok * sizeof(float) == 4096, "partial products of a row block and tile");
  const size_t step = route_tile_step(part_bytes, q.S, q.MB);
  for (size_t t0 = 0; t0 < q.tiles; t0 += step) {
    t.ntile = static_cast<int>(std::min(step, q.tiles - t0));
    t.tok0 = t0 * kTok;
    t.npool = dma && t0 == 0 ? p.B * ncb : 0;
    t.nfold = dma && t0 == 0 ? static_cast<int>(nfold) : 0;
    const unsigned grid = static_cast<unsigned>(static_cast<size_t>(t.ntile) * q.RC * q.S) + t.npool + t.nfold;
    if (dma) launch_products<T, true>(q, p, t, grid, s);
    else launch_products<T, false>(q, p, t, grid, s);
    const size_t left = std::min(static_cast<size_t>(t.ntile) * kTok, N - t.tok0);
    launch_finish<T>(p, t, static_cast<unsigned>((left + 15) / 16), s);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_route_tile(const RouteParams& p, bool bf16, size_t part_bytes, hipStream_t s) {
  const Plan q = make_plan(p, bf16);
  return bf16 ? launch_tile_t<rolesub::bf16>(p, q, part_bytes, s) : launch_tile_t<float>(p, q, part_bytes, s);
}

void launch_pool_any(const RouteParams& p, hipStream_t s) {
  const int ncb = (p.d + 511) / 512, nfb = (p.Hr * p.C + 255) / 256;
  hipLaunchKernelGGL(k_route_pool_any, dim3(static_cast<unsigned>(p.B * ncb + nfb)), dim3(256), 0, s, p);
}

}  // namespace rolesub
