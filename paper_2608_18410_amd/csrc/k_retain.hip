// Token-level retention ahead of the routed path (Sec. 3.1; Sec. 4.1):
// per sample and per segment of consecutive tokens (a camera view), keep the
// highest-scoring tokens, then gather the kept tokens' rows.
#include "common.hpp"
#include "launch.hpp"

namespace rolesub {
namespace {

// Order-preserving unsigned key of a score: a larger score gives a larger
// key, -0 and +0 give the same key, and NaN gives 0, below every number.
__device__ __forceinline__ uint32_t score_key(float x) {
  if (x != x) return 0u;
  const uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// One workgroup per (sample, segment). The keep-th largest key t is found two bits
// at a time from the top: each of 16 steps counts the keys at or above the three
// candidates (ballots, one barrier). Token i is kept when its key is above t, or
// equal to t with fewer than keep - (keys above t) equal keys at lower indices;
// kept tokens are written in index order (block-wide scan of both flags).
// Bound by the chain of steps, at any segment length that occurs: counting each
// token's rank against every other grew with its square. Measured, 128 segments
// of 256: 8.9 -> 7.4 us; of 700: 51 -> 9.4; 64 of 1400: 186 -> 13.4; 4 of 8192:
// 5603 -> 59. A short segment's ranks take less than the chain (128 segments of
// 1, 16, 64, 128: 3.4, 3.6, 4.5, 5.9 us against 7.3), so up to kRankSeg tokens
// are counted, one thread each.
__global__ __launch_bounds__(256) void k_retain(RetainParams p) {
  constexpr int kReg = 4;  // keys per thread in registers; later ones are read from LDS
  constexpr int kRankSeg = 192;
  __shared__ __attribute__((aligned(16))) uint32_t keys[kRetainMaxSeg];
  __shared__ int cnt[2][4][3];
  __shared__ int wgt[2][4], weq[2][4];
  const int b = blockIdx.x / p.n_seg, sg = blockIdx.x % p.n_seg;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n = p.seg_len[sg], start = p.seg_start[sg], keep = p.seg_keep[sg];
  if (keep <= 0) return;
  const float* sc = p.scores + static_cast<size_t>(b) * p.N + start;
  if (n <= kRankSeg) {
    const uint32_t k = tid < n ? score_key(sc[tid]) : 0u;
    keys[tid] = k;  // key 0 at an index past every token ranks before none
    __syncthreads();
    int rank = 0;
    // four keys per 16-byte read; the same address in every lane is a broadcast
#pragma unroll 4
    for (int j = 0; j < n; j += 4) {
      const u32x4 kj = *reinterpret_cast<const u32x4*>(keys + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) rank += (kj[e] > k) | ((kj[e] == k) & (j + e < tid));
    }
    const bool kept = tid < n && rank < keep;
    const uint64_t bal = __ballot(kept);
    if (lane == 0) wgt[0][w] = __popcll(bal);
    __syncthreads();
    int at = __popcll(bal & ((1ull << lane) - 1ull));
    for (int v = 0; v < w; ++v) at += wgt[0][v];
    if (kept) p.keep_idx[static_cast<size_t>(b) * p.K + p.seg_out[sg] + at] = start + tid;
    return;
  }
  uint32_t kr[kReg];
#pragma unroll
  for (int u = 0; u < kReg; ++u) {
    const int i = tid + 256 * u;
    kr[u] = i < n ? score_key(sc[i]) : 0u;  // candidates are above 0: padding is never counted
  }
  for (int i = tid + 256 * kReg; i < n; i += 256) keys[i] = score_key(sc[i]);  // read by this thread only
  uint32_t t = 0;
#pragma unroll 1
  for (int step = 0; step < 16; ++step) {
    const uint32_t one = 1u << (30 - 2 * step);
    int c[3] = {0, 0, 0};
    auto count = [&](uint32_t k) {
#pragma unroll
      for (int j = 0; j < 3; ++j) c[j] += __popcll(__ballot(k >= t + (j + 1) * one));
    };
#pragma unroll
    for (int u = 0; u < kReg; ++u)
      if (256 * u < n) count(kr[u]);
    for (int c0 = 256 * kReg; c0 < n; c0 += 256) count(c0 + tid < n ? keys[c0 + tid] : 0u);
    if (lane == 0)
#pragma unroll
      for (int j = 0; j < 3; ++j) cnt[step & 1][w][j] = c[j];
    __syncthreads();  // (two count buffers: the next step's writes need no second barrier)
    uint32_t up = 0;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const int all = cnt[step & 1][0][j] + cnt[step & 1][1][j] + cnt[step & 1][2][j] + cnt[step & 1][3][j];
      up += all >= keep ? one : 0u;  // the counts fall with j
    }
    t += up;
  }
  // keys above t
  {
    int c = 0;
#pragma unroll
    for (int u = 0; u < kReg; ++u) c += __popcll(__ballot(kr[u] > t));
    for (int c0 = 256 * kReg; c0 < n; c0 += 256) c += __popcll(__ballot((c0 + tid < n ? keys[c0 + tid] : 0u) > t));
    if (lane == 0) cnt[0][w][0] = c;
  }
  __syncthreads();
  const int need = keep - (cnt[0][0][0] + cnt[0][1][0] + cnt[0][2][0] + cnt[0][3][0]);  // equal keys to keep
  int32_t* out = p.keep_idx + static_cast<size_t>(b) * p.K + p.seg_out[sg];
  int base_gt = 0, base_eq = 0;  // keys above and equal to t before this chunk
  const uint64_t below = (1ull << lane) - 1ull;
  auto place = [&](int ch, uint32_t k) {
    const int i = 256 * ch + tid, bf = ch & 1;
    const bool gt = i < n && k > t, eq = i < n && k == t;
    const uint64_t bg = __ballot(gt), be = __ballot(eq);
    if (lane == 0) {
      wgt[bf][w] = __popcll(bg);
      weq[bf][w] = __popcll(be);
    }
    __syncthreads();
    int pg = base_gt + __popcll(bg & below), pe = base_eq + __popcll(be & below);
    for (int v = 0; v < 4; ++v) {
      pg += v < w ? wgt[bf][v] : 0;
      pe += v < w ? weq[bf][v] : 0;
      base_gt += wgt[bf][v];
      base_eq += weq[bf][v];
    }
    if (gt || (eq && pe < need)) out[pg + min(pe, need)] = start + i;
  };
#pragma unroll
  for (int u = 0; u < kReg; ++u)
    if (256 * u < n) place(u, kr[u]);
  for (int ch = kReg; 256 * ch < n; ++ch) place(ch, 256 * ch + tid < n ? keys[256 * ch + tid] : 0u);
}

// dst[b, j, :] = src[b, idx[b, j], :], rows of row_bytes (a multiple of 4).
// One workgroup per (sample, kept token); 16-byte pieces when row_bytes allows.
// An index outside [0, N) falls outside the sample's buffer resource and
// gives a zero row.
__global__ __launch_bounds__(256) void k_gather_rows(GatherParams p) {
  const size_t row = blockIdx.x;
  const int b = static_cast<int>(row / p.K);
  const int32_t t = p.idx[row];
  const uint32_t rb = static_cast<uint32_t>(p.row_bytes);
  const rsrc_t r_src = make_rsrc(static_cast<const char*>(p.src) + static_cast<size_t>(b) * p.N * p.row_bytes,
                                 clamp_bytes(static_cast<size_t>(p.N) * p.row_bytes));
  const rsrc_t r_dst = make_rsrc(static_cast<char*>(p.dst) + row * p.row_bytes, rb);
  const bool in = (t >= 0) & (t < p.N);
  const uint32_t so = in ? static_cast<uint32_t>(t) * rb : kOOB;
  if ((rb & 15u) == 0) {
    // four 16-byte loads in flight per thread before their stores
    for (uint32_t o0 = 16u * threadIdx.x; o0 < rb; o0 += 4u * 16u * 256u) {
      u32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t o = o0 + u * 16u * 256u;
        v[u] = bload16(r_src, (so == kOOB) | (o >= rb) ? kOOB : so + o);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t o = o0 + u * 16u * 256u;
        __builtin_amdgcn_raw_buffer_store_b128(v[u], r_dst, o < rb ? o : kOOB, 0, 0);
      }
    }
  } else {
    for (uint32_t o = 4u * threadIdx.x; o < rb; o += 4u * 256u) {
      const uint32_t v = bload4(r_src, so == kOOB ? kOOB : so + o);
      __builtin_amdgcn_raw_buffer_store_b32(v, r_dst, o, 0, 0);
    }
  }
}

}  // namespace

hipError_t launch_retain(const RetainParams& p, hipStream_t s) {
  if (p.B == 0 || p.n_seg == 0 || p.K == 0) return hipSuccess;
  hipLaunchKernelGGL(k_retain, dim3(static_cast<unsigned>(p.B * p.n_seg)), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_gather_rows(const GatherParams& p, hipStream_t s) {
  if (p.B == 0 || p.K == 0 || p.row_bytes == 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_rows, dim3(static_cast<unsigned>(static_cast<size_t>(p.B) * p.K)), dim3(256), 0, s,
                     p);
  return hipGetLastError();
}

}  // namespace rolesub
