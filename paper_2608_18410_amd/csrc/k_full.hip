// Full-width routing space (Sec. 3.2 with one R over the whole value vector,
// d_v = H*dh; Sec. 4.1 runs d_v = 4096 with S = 16 groups of 256).
//
// Tokens that keep all S groups have R M R^T v = v, so the cache holds their
// value vector (S consecutive slots = d_v contiguous values). Routed tokens
// (any other mask) go through two dense contractions on the bf16 matrix cores:
//   rotate:  z  = R^T v  for every routed token, only the kept groups stored;
//   values:  v~ = R z~   for every routed token, written head-major
//            [B][H][T][dh] for the attention kernel.
// Both are one gather-GEMM C[m][n] = sum_k A[m][k] * Bt[n][k] over the routed
// tokens of all samples (m), with Bt = R^T (rotate; the caller supplies the
// transpose of the frozen R) or Bt = R (values), so that both operands are
// read along k. A routed-token list per sample and the cache offsets come from
// a small preparation kernel.
#include "common.hpp"
#include "launch.hpp"

namespace rolesub {
namespace {

constexpr int kBN = 128, kBK = 64;  // columns of a tile, k per stage
constexpr int kPrepChunks = 16;

__device__ __forceinline__ uint32_t full_bits(int S) { return S >= 32 ? 0xFFFFFFFFu : ((1u << S) - 1u); }

// Inclusive scan over the 64 lanes of a wave.
__device__ __forceinline__ int wave_incl_scan(int x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  return x;
}

// Per sample: the routed-token list (and its length), the cache offsets
// (PACK), and the value-space copies of the tokens that keep every group:
// into the cache (PACK: v -> Vp) or from it into the head-major values
// (!PACK: Vp -> Vh, at the given offsets). kPrepChunks workgroups per sample
// share the copies; the first one writes the list, count and offsets, and
// (PACK) workgroup c builds the per-group lists of groups c, c + kPrepChunks.
template <bool PACK>
__global__ __launch_bounds__(256) void k_full_prep(FullParams p) {
  // offsets, the value-space token list and (PACK) the masks of the sample,
  // sized by T at launch (prep_shm)
  extern __shared__ __attribute__((aligned(16))) char prep_smem[];
  int* s_off = reinterpret_cast<int*>(prep_smem);
  uint32_t* s_mask = reinterpret_cast<uint32_t*>(prep_smem + 4 * (p.T + 1));
  uint16_t* s_full = reinterpret_cast<uint16_t*>(prep_smem + 4 * (p.T + 1) + (PACK ? 4 * p.T : 0));
  __shared__ int wtot[4], wfull[4];
  __shared__ int wcnt[4][32];
  const int b = blockIdx.x / kPrepChunks, chunk = blockIdx.x % kPrepChunks;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int T = p.T, S = p.S;
  const uint32_t full = full_bits(S);
  const uint32_t* mk = p.mask + static_cast<size_t>(b) * T;
  int run_pc = 0, run_rt = 0, run_full = 0;
  for (int c0 = 0; c0 < T; c0 += 256) {
    const int t = c0 + tid;
    const bool valid = t < T;
    const uint32_t m = valid ? (mk[t] & full) : 0u;
    const bool routed = valid && m != full, isfull = valid && m == full;
    // packed scan: kept-group count (low 16 bits, at most 256 * 32 per
    // chunk) and routed flag (high bits); full tokens by ballot
    const int x = (valid ? __popc(m) : 0) | (routed ? (1 << 16) : 0);
    const int inc = wave_incl_scan(x);
    const uint64_t bal = __ballot(isfull);
    if (lane == 63) wtot[w] = inc;
    if (lane == 0) wfull[w] = __popcll(bal);
    __syncthreads();
    int before = 0, before_full = 0;
    for (int v = 0; v < w; ++v) {
      before += wtot[v];
      before_full += wfull[v];
    }
    const int ex = before + inc - x;
    const int ex_pc = ex & 0xFFFF, ex_rt = ex >> 16;
    const int ex_full = before_full + __popcll(bal & ((1ull << lane) - 1ull));
    if (valid) s_off[t] = run_pc + ex_pc;
    if (PACK && valid) s_mask[t] = m;
    if (chunk == 0 && routed) p.rlist[static_cast<size_t>(b) * T + run_rt + ex_rt] = t;
    if (isfull) s_full[run_full + ex_full] = static_cast<uint16_t>(t);
    const int tot = wtot[0] + wtot[1] + wtot[2] + wtot[3];
    run_pc += tot & 0xFFFF;
    run_rt += tot >> 16;
    run_full += wfull[0] + wfull[1] + wfull[2] + wfull[3];
    __syncthreads();
  }
  if (chunk == 0) {
    if (tid == 0) p.counts[b] = run_rt;
    if (PACK) {
      int32_t* off = p.offsets + static_cast<size_t>(b) * (T + 1);
      for (int t = tid; t < T; t += 256) off[t] = s_off[t];
      if (tid == 0) off[T] = run_pc;
    }
  }
  if (PACK) {
    // Per group: the routed tokens that keep it, in token order, after the
    // earlier groups' lists. Every workgroup of the sample counts every
    // group's tokens (one ballot per group per 256 tokens) and then lists
    // the tokens of its own groups (chunk, chunk + kPrepChunks).
    int32_t* pr = p.pairs + static_cast<size_t>(b) * T * S;
    int run_g[32];
#pragma unroll
    for (int gg = 0; gg < 32; ++gg) run_g[gg] = 0;
    for (int c0 = 0; c0 < T; c0 += 256) {
      const int t = c0 + tid;
      const uint32_t m = t < T ? s_mask[t] : full;
      const uint32_t kept = m != full ? m : 0u;
#pragma unroll
      for (int gg = 0; gg < 32; ++gg) {
        if (gg < S) {
          const uint64_t bal = __ballot((kept >> gg) & 1u);
          if (lane == 0) wcnt[w][gg] = __popcll(bal);
        }
      }
      __syncthreads();
#pragma unroll
      for (int gg = 0; gg < 32; ++gg)
        if (gg < S) run_g[gg] += wcnt[0][gg] + wcnt[1][gg] + wcnt[2][gg] + wcnt[3][gg];
      __syncthreads();
    }
    for (int g = chunk; g < S; g += kPrepChunks) {
      int start = 0;
#pragma unroll
      for (int gg = 0; gg < 32; ++gg) start += gg < g ? run_g[gg] : 0;
      int n_g = 0;
#pragma unroll
      for (int gg = 0; gg < 32; ++gg) n_g = gg == g ? run_g[gg] : n_g;
      if (tid == 0) {
        p.counts_g[static_cast<size_t>(b) * S + g] = n_g;
        p.starts_g[static_cast<size_t>(b) * S + g] = start;
      }
      int run = start;
      for (int c0 = 0; c0 < T; c0 += 256) {
        const int t = c0 + tid;
        const uint32_t m = t < T ? s_mask[t] : full;
        const bool keeps = m != full && ((m >> g) & 1u);
        const uint64_t bal = __ballot(keeps);
        if (lane == 0) wtot[w] = __popcll(bal);
        __syncthreads();
        int o = run + __popcll(bal & ((1ull << lane) - 1ull));
        for (int v = 0; v < w; ++v) o += wtot[v];
        if (keeps) pr[o] = t;
        run += wtot[0] + wtot[1] + wtot[2] + wtot[3];
        __syncthreads();
      }
    }
  }
  // value-space copies of the full tokens: d_v/8 16-byte pieces each, work
  // items (token, piece) spread over the chunks' threads, 8 loads in flight.
  const int pieces = p.dv / 8, dh = p.dv / p.H;
  const int cc = chunk, ncc = kPrepChunks;
  const int n_items = run_full * pieces;
  const rsrc_t r_cache = make_rsrc(static_cast<const bf16*>(p.Vp) + static_cast<size_t>(b) * p.cap * p.ds,
                                   clamp_bytes(static_cast<size_t>(p.cap) * p.ds * 2));
  const rsrc_t r_v = make_rsrc(static_cast<const bf16*>(p.v) + static_cast<size_t>(b) * T * p.dv,
                               clamp_bytes(static_cast<size_t>(T) * p.dv * 2));
  const int32_t* goff = p.offsets + static_cast<size_t>(b) * (T + 1);
  for (int i0 = (cc * 256 + tid); i0 < n_items; i0 += 8 * 256 * ncc) {
    u32x4 val[8];
    int tok[8], pc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * 256 * ncc;
      const bool ok = i < n_items;
      tok[u] = ok ? s_full[i / pieces] : 0;
      pc[u] = i % pieces;
      uint32_t src;
      if (PACK) {
        src = oob_unless(ok, static_cast<uint32_t>((tok[u] * p.dv + 8 * pc[u]) * 2));
        val[u] = bload16(r_v, src);
      } else {
        // the piece lies in slot o + 8 pc / ds of the token's S consecutive slots
        const int o = ok ? goff[tok[u]] : 0;
        const bool in_cap = o + (8 * pc[u]) / p.ds < p.cap;
        src = oob_unless(ok && in_cap, static_cast<uint32_t>((static_cast<size_t>(o) * p.ds + 8 * pc[u]) * 2));
        val[u] = bload16(r_cache, src);
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * 256 * ncc;
      if (i >= n_items) continue;
      if (PACK) {
        const int o = s_off[tok[u]];
        if (o + (8 * pc[u]) / p.ds < p.cap) {
          bf16* dst = static_cast<bf16*>(p.Vp) + (static_cast<size_t>(b) * p.cap + o) * p.ds + 8 * pc[u];
          *reinterpret_cast<u32x4*>(dst) = val[u];
        }
      } else {
        const int e = 8 * pc[u], h = e / dh;
        bf16* dst = static_cast<bf16*>(p.Vh) + ((static_cast<size_t>(b) * p.H + h) * T + tok[u]) * dh + (e - h * dh);
        *reinterpret_cast<u32x4*>(dst) = val[u];
      }
    }
  }
}

// C[m][n] = sum_k A[m][k] * Bt[n][k] on 16x16x32 bf16 MFMA, a TBM x 128 tile per
// workgroup, waves of (TBM / WM) x 64, k in stages of 64.
//   MODE 0 (rotate): rows are the routed tokens of all samples that keep the
//   workgroup's group g (per-sample lists from the preparation kernel), so only
//   kept groups are computed; A = v, Bt = the rows of R^T for group g's output
//   dims; results to the cache.
//   MODE 1 (values): rows are the routed tokens of all samples; A = their cached
//   groups of z~ (zero where dropped; stages of groups that no row of the tile
//   keeps are skipped), Bt = R; results head-major.
// Rows map to (sample, token) through the prefix of the per-sample counts.
// Groups (MODE 0) or column tiles (MODE 1) are pinned to XCDs so that each XCD
// reads only its share of R into its L2.
//
// Buffer->LDS DMA brings the stages into a ring of RING (operands in flight in
// registers, two sets of them at most, covered little of the round trip to L2).
// Rows of 128 bytes, 16-byte chunks XOR-swizzled by row pair (conflict-free
// fragment reads). One barrier per stage. NCP = 0: every wave issues its share of
// the DMAs between its MFMAs. NCP > 0: NCP waves do nothing else, since a wave whose
// DMA waits for the texture unit holds up the MFMAs behind it.
// Operands off 16-byte boundaries (DMA = false) go through registers instead, two
// stages in flight, and two LDS buffers (see the loop).
// Bound by the texture unit, which takes a 128-byte line of a DMA in about 2.6
// clocks, and for the 256-row tile by that and the MFMAs in turn (a wave that
// only touches later lines to bring them into L2 made both slower, 52 -> 79 us).
//
// Measured at d_v = 4096, 64 prefixes of 81 tokens, 32 of them routed, preparation
// included, against register staging:
//   rotate, 4 (8, 15) of 16 groups kept: 73.5 (99.6, 120.6) -> 52.4 (75, 93) us with 64 rows,
//     three stages, two workgroups per CU; six stages and one per CU: 62 (a group's
//     last row tile then starts when the others end); with copying waves: 59;
//   values, 256 rows, eight MFMA and four copying waves: 105 -> 78 us; no
//     copying waves: 87; 128 rows: 97-118; 64 rows: 121. One prefix (16), 64 rows:
//     65 (70) -> 37 (41) us, 256 rows: 54 (57). A values product over each group's kept
//     rows only, with f32 accumulators in LDS, took 140 us (uncoalesced fragments).
//   Off 16-byte boundaries, 8 (2) bytes off, preparation included, against the
//     register staging before the DMA rings: rotate 69.5 (68) -> 60 (73) us at 64
//     prefixes, 44 (44) -> 36.5 (38) at one; values, 128 rows as there, 98 (101) -> 89
//     (93) and 67 (67) -> 58 (59.5). Loaded and stored at once, nothing in flight: 147
//     (151), 120 (122), 284 (288) and 119 (120).
__device__ __forceinline__ int full_swz(int row) { return (row >> 1) & 7; }

template <int MODE, int TBM, int WM, int RING, int NWG, int NCP, bool DMA = true>
__global__ __launch_bounds__(128 * WM + 64 * NCP, (NWG * (2 * WM + NCP) + 3) / 4) void k_full_gemm(FullParams p) {
  constexpr int NW = 2 * WM, NT = 64 * NW, NP = NCP ? NCP : NW, MI = TBM / WM / 16;  // MFMA waves, their threads, copying waves, 16-row blocks per wave
  constexpr int kStA = TBM * kBK * 2, kStB = kBN * kBK * 2, kStage = kStA + kStB;  // bytes
  constexpr int UA = kStA / 1024 / NP, UB = kStB / 1024 / NP;  // A and B DMAs per copying wave and stage
  static_assert(kBK == 64 && kStA % (1024 * NP) == 0 && kStB % (1024 * NP) == 0 && (DMA ? RING >= 3 : RING == 2 && NCP == 0),
                "stage shape");
  __shared__ __attribute__((aligned(16))) char ring[RING * kStage];
  __shared__ int pre[kFullMaxB + 1];
  __shared__ int r_b[TBM], r_t[TBM], r_off[TBM];
  __shared__ uint32_t r_mask[TBM];
  __shared__ uint32_t s_or;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, g4 = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int B = p.B, T = p.T, dv = p.dv, S = p.S, ds = p.ds;
  // which tile: (group g, column sub-tile, row tile) or (column tile, row tile)
  int g = 0, n0, mt;
  if (MODE == 0) {
    const int nsub = ds / kBN;
    int rest;
    xcd_split(blockIdx.x, S, g, rest);
    n0 = g * ds + (rest % nsub) * kBN;
    mt = rest / nsub;
  } else {
    int nt;
    xcd_split(blockIdx.x, dv / kBN, nt, mt);
    n0 = nt * kBN;
  }
  const int m0 = mt * TBM;

  // prefix over samples of the row counts (one wave, 64 samples per step)
  if (w == 0) {
    int run = 0;
    for (int c0 = 0; c0 < B; c0 += 64) {
      const int x = c0 + lane < B ? (MODE == 0 ? p.counts_g[static_cast<size_t>(c0 + lane) * S + g]
                                               : p.counts[c0 + lane]) : 0;
      const int inc = wave_incl_scan(x);
      if (c0 + lane < B) pre[c0 + lane] = run + inc - x;
      run += __shfl(inc, 63, kWave);
    }
    if (lane == 0) pre[B] = run;
  }
  if (tid == 0) s_or = 0;
  __syncthreads();
  const int total = pre[B];
  if (m0 >= total) return;  // the same in every thread
  if (tid < TBM) {
    const int r = m0 + tid;
    int bb = -1, tt = 0, oo = 0;
    uint32_t mm = 0;
    if (r < total) {
      int lo = 0, hi = B - 1;  // largest bb with pre[bb] <= r
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= r) lo = mid; else hi = mid - 1;
      }
      bb = lo;
      const int j = r - pre[bb];
      tt = MODE == 0 ? p.pairs[static_cast<size_t>(bb) * T * S + p.starts_g[static_cast<size_t>(bb) * S + g] + j]
                     : p.rlist[static_cast<size_t>(bb) * T + j];
      mm = p.mask[static_cast<size_t>(bb) * T + tt] & full_bits(S);
      oo = p.offsets[static_cast<size_t>(bb) * (T + 1) + tt];
      if (MODE == 1) atomicOr(&s_or, mm);
    }
    r_b[tid] = bb;
    r_t[tid] = tt;
    r_mask[tid] = mm;
    r_off[tid] = oo;
  }
  __syncthreads();
  const uint32_t tile_or = MODE == 1 ? __builtin_amdgcn_readfirstlane(s_or) : full_bits(S);

  // DMA j of an operand fills its LDS bytes 1024 j ..: rows 8j .. 8j + 7, lane
  // i's 16 bytes at row 8j + i / 8, position i % 8, which holds chunk
  // (i % 8) ^ full_swz(row). Copying wave pw issues DMAs pw, pw + NP, ...
  const int pw = NCP ? max(w - NW, 0) : w;  // (unused in MFMA waves of NCP > 0)
  const rsrc_t r_A = MODE == 0
      ? make_rsrc(p.v, clamp_bytes(static_cast<size_t>(B) * T * dv * 2))
      : make_rsrc(p.Vp, clamp_bytes(static_cast<size_t>(B) * p.cap * ds * 2));
  const rsrc_t r_B = make_rsrc(p.Rm, clamp_bytes(static_cast<size_t>(dv) * dv * 2));
  // A rows: MODE 0 the byte offset of the token's value row, MODE 1 the byte
  // offset of the sample's cache and the token's mask and first slot
  uint32_t a_base[UA], a_mask[UA], b_base[UB];
  int a_slot0[UA];
  bool a_ok[UA];
#pragma unroll
  for (int u = 0; u < UA; ++u) {
    const int row = 8 * (pw + NP * u) + (lane >> 3), bb = r_b[row];
    const uint32_t ch = 16u * ((lane & 7) ^ full_swz(row));
    a_ok[u] = bb >= 0;
    a_mask[u] = r_mask[row];
    a_slot0[u] = r_off[row];
    a_base[u] = ch + (MODE == 0 ? static_cast<uint32_t>((static_cast<size_t>(bb < 0 ? 0 : bb) * T + r_t[row]) * dv * 2)
                                : static_cast<uint32_t>(static_cast<size_t>(bb < 0 ? 0 : bb) * p.cap * ds * 2));
  }
#pragma unroll
  for (int u = 0; u < UB; ++u) {
    const int row = 8 * (pw + NP * u) + (lane >> 3);
    b_base[u] = static_cast<uint32_t>(static_cast<size_t>(n0 + row) * dv * 2) + 16u * ((lane & 7) ^ full_swz(row));
  }
  const int cap32 = static_cast<int>(p.cap);  // < 2^31: a sample's cache is < 2 GiB
  const uint32_t ring_base = lds_addr(ring);
  // k of the stages: every stage of every group in tile_or (MODE 0: all groups);
  // past the last, k stays at dv and the DMAs are out of range (they write zeros
  // to a free stage), so the number of pending ones stays known
  auto next_k = [&](int k0) -> int {
    const int k1 = k0 + kBK;
    if (k0 >= dv) return dv;
    if (MODE == 0 || k1 % ds != 0) return k1;
    const int gb = k1 / ds;
    const uint32_t rest = gb < 32 ? (tile_or >> gb) : 0u;
    return rest ? (gb + static_cast<int>(__builtin_ctz(rest))) * ds : dv;
  };
  int kq = tile_or == 0 ? dv : static_cast<int>(__builtin_ctz(tile_or)) * ds;
  const int nst = MODE == 0 ? dv / kBK : __popc(tile_or) * (ds / kBK);
  // piece u (A pieces, then B) at k0: copied from, to (the wave's 1024 bytes at)
  auto piece = [&](int k0, int u, auto&& copy) {
    const bool real = k0 < dv;
    if (u < UA) {
      uint32_t off;
      bool ok = real & a_ok[u];
      if (MODE == 0) {
        off = a_base[u] + 2u * k0;
      } else {
        const int gk = min(k0 / ds, 31);
        const int slot = a_slot0[u] + __popc(a_mask[u] & ((1u << gk) - 1u));
        ok = ok & ((a_mask[u] >> gk) & 1u) & (slot < cap32);
        off = a_base[u] + static_cast<uint32_t>((slot * ds + (k0 - gk * ds)) * 2);
      }
      copy(r_A, oob_unless(ok, off), 1024u * (pw + NP * u));
    } else {
      copy(r_B, oob_unless(real, b_base[u - UA] + 2u * k0), kStA + 1024u * (pw + NP * (u - UA)));
    }
  };
  auto issue = [&](int buf, int k0, int u) {
    const uint32_t dst = buf * kStage;
    piece(k0, u, [&](rsrc_t r, uint32_t off, uint32_t to) { dma16(r, off, ring_base + (dst + to)); });
  };
  auto fill_ring = [&]() {
#pragma unroll
    for (int s = 0; s < RING; ++s) {
#pragma unroll
      for (int u = 0; u < UA + UB; ++u) issue(s, kq, u);
      kq = next_k(kq);
    }
    wait_vmcnt<(UA + UB) * (RING - 1)>();  // the first stage
  };
  if (NCP && w >= NW) {
    // copying wave: the barriers of the MFMA waves, below
    fill_ring();
    __syncthreads();
    for (int s = 0, cur = 0; s < nst; ++s) {
      wait_vmcnt<(UA + UB) * (RING - 2)>();  // stage s + 1: RING - 2 younger ones may be pending
      __syncthreads();
#pragma unroll
      for (int u = 0; u < UA + UB; ++u) issue(cur, kq, u);
      kq = next_k(kq);
      cur = cur + 1 == RING ? 0 : cur + 1;
    }
    wait_vmcnt<0>();  // trailing out-of-range DMAs land before the ring is reused
    __syncthreads();
    __syncthreads();
    return;
  }
  if (!NCP && DMA) fill_ring();

  f32x4 acc[MI][4];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int wm = w >> 1, wn = w & 1;
  struct Frags {
    bf16x8 a[MI], b[4];
  };
  auto read = [&](Frags& f, int buf, int ks) {
    const char* st = ring + buf * kStage;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int r = (TBM / WM) * wm + 16 * i + l16;
      f.a[i] = *reinterpret_cast<const bf16x8*>(st + r * 128 + 16 * ((4 * ks + g4) ^ full_swz(r)));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = 64 * wn + 16 * j + l16;
      f.b[j] = *reinterpret_cast<const bf16x8*>(st + kStA + r * 128 + 16 * ((4 * ks + g4) ^ full_swz(r)));
    }
  };
  // A stage's two MFMA k-steps run one half stage behind their fragment reads.
  Frags f0, f1;
  if constexpr (DMA) {
    // When every wave has read a stage's second half (the barrier in its middle),
    // the DMAs of the stage RING further on refill its buffer, spread between MFMAs.
    __syncthreads();
    read(f0, 0, 0);
    int cur = 0;
    for (int s = 0; s < nst; ++s) {
      read(f1, cur, 1);
#pragma unroll
      for (int q = 0; q < 4 * MI; ++q) acc[q / 4][q % 4] = mfma_16x16x32(f0.a[q / 4], f0.b[q % 4], acc[q / 4][q % 4]);
      if (!NCP) wait_vmcnt<(UA + UB) * (RING - 2)>();  // as a copying wave
      __syncthreads();
      const int nxt = cur + 1 == RING ? 0 : cur + 1;
      read(f0, nxt, 0);
#pragma unroll
      for (int q = 0; q < 4 * MI; ++q) {
        acc[q / 4][q % 4] = mfma_16x16x32(f1.a[q / 4], f1.b[q % 4], acc[q / 4][q % 4]);
#pragma unroll
        for (int u = 0; u < UA + UB; ++u)
          if (!NCP && u * 4 * MI / (UA + UB) == q) issue(cur, kq, u);
      }
      if (!NCP) kq = next_k(kq);
      cur = nxt;
    }
  } else {
    // Two register sets, each loaded two stages before it is stored, and two
    // buffers: at the barrier in the middle of a stage the next one is in LDS and
    // the one before it has been read. An even number of stages (ds is a multiple
    // of 128).
    struct Regs {
      u32x4 v[UA + UB];
    };
    auto load = [&](Regs& x) {
#pragma unroll
      for (int u = 0; u < UA + UB; ++u) piece(kq, u, [&](rsrc_t r, uint32_t off, uint32_t) { x.v[u] = bload16(r, off); });
      kq = next_k(kq);
    };
    auto store = [&](const Regs& x, int buf) {
#pragma unroll
      for (int u = 0; u < UA + UB; ++u) {
        const int to = u < UA ? 1024 * (pw + NP * u) : kStA + 1024 * (pw + NP * (u - UA));
        *reinterpret_cast<u32x4*>(ring + buf * kStage + to + 16 * lane) = x.v[u];
      }
    };
    auto step = [&](Regs& x, int cur) {
      read(f1, cur, 1);
#pragma unroll
      for (int q = 0; q < 4 * MI; ++q) acc[q / 4][q % 4] = mfma_16x16x32(f0.a[q / 4], f0.b[q % 4], acc[q / 4][q % 4]);
      store(x, cur ^ 1);
      load(x);
      __syncthreads();
      read(f0, cur ^ 1, 0);
#pragma unroll
      for (int q = 0; q < 4 * MI; ++q) acc[q / 4][q % 4] = mfma_16x16x32(f1.a[q / 4], f1.b[q % 4], acc[q / 4][q % 4]);
    };
    Regs ra, rb;
    load(ra);
    load(rb);
    store(ra, 0);
    load(ra);
    __syncthreads();
    read(f0, 0, 0);
    for (int s = 0; s < nst; s += 2) {
      step(rb, 0);
      step(ra, 1);
    }
  }
  wait_vmcnt<0>();  // as a copying wave
  __syncthreads();

  // stage the bf16 tile in LDS (row stride kBN + 8), then 16-byte stores
  constexpr int kCs = kBN + 8;
  static_assert(TBM * kCs * 2 <= RING * kStage, "C tile fits the ring");
  bf16* Cs = reinterpret_cast<bf16*>(ring);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        Cs[((TBM / WM) * wm + 16 * i + 4 * g4 + e) * kCs + 64 * wn + 16 * j + l16] = static_cast<bf16>(acc[i][j][e]);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < TBM * kBN / 8 / NT; ++u) {
    const int q = tid + NT * u, row = q / (kBN / 8), c = q % (kBN / 8);
    const int bb = r_b[row];
    if (bb < 0) continue;
    const u32x4 val = *reinterpret_cast<const u32x4*>(&Cs[row * kCs + 8 * c]);
    const int n = n0 + 8 * c;
    if (MODE == 0) {
      const uint32_t mm = r_mask[row];
      const int slot = r_off[row] + __popc(mm & ((1u << g) - 1u));
      if (slot < p.cap) {
        bf16* dst = static_cast<bf16*>(p.Vp) + (static_cast<size_t>(bb) * p.cap + slot) * ds + (n - g * ds);
        *reinterpret_cast<u32x4*>(dst) = val;
      }
    } else {
      const int dh = dv / p.H, h = n / dh;
      bf16* dst = static_cast<bf16*>(p.Vh) + ((static_cast<size_t>(bb) * p.H + h) * T + r_t[row]) * dh + (n - h * dh);
      *reinterpret_cast<u32x4*>(dst) = val;
    }
  }
}

// Rt[j][k] = R[k][j] for an n x n bf16 matrix, 64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void k_transpose_bf16(const bf16* __restrict__ R, bf16* __restrict__ Rt, int n) {
  __shared__ bf16 tile[64][66];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int bx = blockIdx.x % (n / 64), by = blockIdx.x / (n / 64);
  for (int r = ty; r < 64; r += 4) tile[r][tx] = R[static_cast<size_t>(by * 64 + r) * n + bx * 64 + tx];
  __syncthreads();
  for (int r = ty; r < 64; r += 4) Rt[static_cast<size_t>(bx * 64 + r) * n + by * 64 + tx] = tile[tx][r];
}

}  // namespace

hipError_t launch_full(const FullParams& p, int mode, hipStream_t s) {
  if (p.B == 0 || p.T == 0) return hipSuccess;
  const dim3 gprep(static_cast<unsigned>(p.B) * kPrepChunks);
  const size_t shm_pack = 4 * static_cast<size_t>(p.T + 1) + 4 * static_cast<size_t>(p.T) + 2 * static_cast<size_t>(p.T);
  const size_t shm_vals = 4 * static_cast<size_t>(p.T + 1) + 2 * static_cast<size_t>(p.T);
  // row tiles: at most every token of every sample is a row (upper bound;
  // tiles past the actual count return at once). Values: 256-row tiles need many
  // rows to fill the chip. At 81 tokens a sample, 32 of them routed, the product of
  // 64-row and 256-row tiles took 37 and 54 us for 1 sample, 41 and 57 for 16, 56
  // and 59 for 20, 60 and 61 for 32, 84 and 62 for 40; the line lies lower than the
  // crossing because more of the tokens may be routed.
  const size_t rows = static_cast<size_t>(p.B) * p.T;
  const unsigned ncol = static_cast<unsigned>(p.dv / kBN);
  auto tiles = [&](int tbm) { return dim3(ncol * static_cast<unsigned>((rows + tbm - 1) / tbm)); };
  const void* src = mode == 0 ? p.v : p.Vp;
  const bool dma = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(p.Rm)) & 15) == 0;
  if (mode == 0) {
    hipLaunchKernelGGL(k_full_prep<true>, gprep, dim3(256), shm_pack, s, p);
    if (dma) hipLaunchKernelGGL((k_full_gemm<0, 64, 2, 3, 2, 0>), tiles(64), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((k_full_gemm<0, 64, 2, 2, 2, 0, false>), tiles(64), dim3(256), 0, s, p);
  } else {
    hipLaunchKernelGGL(k_full_prep<false>, gprep, dim3(256), shm_vals, s, p);
    if (!dma) hipLaunchKernelGGL((k_full_gemm<1, 128, 2, 2, 2, 0, false>), tiles(128), dim3(256), 0, s, p);
    else if (rows <= 1536) hipLaunchKernelGGL((k_full_gemm<1, 64, 2, 3, 2, 0>), tiles(64), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((k_full_gemm<1, 256, 4, 3, 1, 4>), tiles(256), dim3(768), 0, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_transpose(const void* R, void* Rt, int n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_transpose_bf16, dim3(static_cast<unsigned>((n / 64) * (n / 64))), dim3(256), 0, s,
                     static_cast<const bf16*>(R), static_cast<bf16*>(Rt), n);
  return hipGetLastError();
}

}  // namespace rolesub
