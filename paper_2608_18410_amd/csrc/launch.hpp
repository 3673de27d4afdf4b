// Internal launcher interface between the C-ABI layer and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rolesub {

struct RouteParams {
  int B, T, d, G, C, d_e, Hr, kind;
  float alpha_role, alpha_lang;
  const void* h;
  const uint8_t* types;
  const void *W_r, *b_r, *E, *W1, *b1, *W2, *b2;
  const void *W_tok, *b_tok, *W_role, *W_lang, *b_lang;
  float* cb;  // [B][Hr or G] per-sample language term (workspace)
  float* F;   // [Hr or G][C] folded role term (workspace)
  float* hbar;  // [B][d] pooled language state (workspace)
  float* pcb;   // [ncb][B][route_ld(Hr or G)] language terms per column block (workspace)
  float* rpart;  // split-K router: both halves' partial products per 96-token tile, or null (workspace)
  int* rcnt;     // split-K router: finished halves per tile, zeroed by the pool kernel (workspace)
  float* part;   // two-kernel form: folded operands and partial products (workspace)
  int sk_polls;  // split-K router: polls the first half of a tile makes for the second (0: never shares)
  int mode;
  int k_by_type[4];
  float tau;
  int kmin, kmax;
  const float* scores_in;
  float* scores_out;
  const void* w_pri;  // [C] role priority weights (call dtype), with priority
  float* priority;    // [B][T] p = w^T a, or null
  uint32_t* mask;     // null: scores (and priority) only, no selection
  uint8_t* idx;
  uint8_t* count;
};

// Row stride (floats) of the per-sample language terms: whole 16-byte pieces.
__host__ __device__ inline size_t route_ld(int n) { return n < 1 ? 0 : (static_cast<size_t>(n) + 3) & ~size_t{3}; }
// Sizes of the route workspace pieces (floats).
inline size_t route_cb_floats(int B, int Hr, int G, int kind) {
  return static_cast<size_t>(B) * route_ld(kind == 0 ? Hr : G);
}
inline size_t route_F_floats(int Hr, int G, int C, int kind) {
  return static_cast<size_t>(kind == 0 ? Hr : G) * C;
}
inline size_t route_hbar_floats(int B, int d) { return static_cast<size_t>(B) * d; }
// column blocks of 256 (the smallest block the pool kernel uses, f32) bound
// the number of partial language terms for any dtype
inline size_t route_pcb_floats(int B, int d, int Hr, int G, int kind) {
  return static_cast<size_t>((d + 255) / 256) * B * route_ld(kind == 0 ? Hr : G);
}

// Split-K form of the bf16 MLP2 router (Hr = 128): 96-token tiles, each
// computed by two workgroups over half of the hidden size.
constexpr int kRouteSkTok = 96;
// shortest prefix the split form takes: a tile then touches at most three samples
constexpr int kRouteSkMinT = kRouteSkTok / 2;
inline size_t route_sk_tiles(int B, int T) { return (static_cast<size_t>(B) * T + kRouteSkTok - 1) / kRouteSkTok; }
// floats of both halves' partials (144 products per token) and ints of the tile counters
inline size_t route_sk_part_floats(int B, int T, int Hr, int kind) {
  return kind == 0 && Hr == 128 ? route_sk_tiles(B, T) * 2 * kRouteSkTok * 144 : 0;
}
// Whether its kernel's 32-bit offsets reach all of its partial products (up to
// 1.86 million tokens); larger calls run the single kernel, in the same bits.
inline bool route_sk_fits(int B, int T) {
  return route_sk_tiles(B, T) * 2 * kRouteSkTok * 144 * sizeof(float) < (size_t{1} << 31);
}
inline size_t route_sk_cnt_ints(int B, int T, int Hr, int kind) {
  return kind == 0 && Hr == 128 ? route_sk_tiles(B, T) : 0;
}

// Two-kernel form (k_route_tile.hip): 64-token tiles x row blocks x slices of
// the hidden size. MB: 16-row blocks of the router's matrices in all.
inline int route_tile_blocks(int Hr, int G, int C, int kind) {
  auto blocks = [](int n) { return n < 1 ? 0 : (n - 1) / 16 + 1; };
  const int MB = blocks(kind == 0 ? Hr : G) + blocks(C);
  return MB < 1 ? 1 : MB;  // sizes are asked for before the router is checked
}
inline int route_tile_rows(int MB) { return MB <= 2 ? 2 : 3; }  // row blocks per workgroup
// Slices of the hidden size: the same for every batch, so that a token's sums
// do not depend on which others share the call. bf16 MLP2: the two halves the
// one-kernel forms sum. Otherwise what fills the chip over the range of batches
// (additive, at most five row blocks: 4; f32, whose stages take four times the
// matrix-core time: 8), with the partial products of a tile within 2 MiB and a
// stage at least in every slice.
inline int route_tile_smax(int MB, int want) {
  const size_t n = (size_t{2} << 20) / (static_cast<size_t>(MB) * 4096);
  return n < 1 ? 1 : n > static_cast<size_t>(want) ? want : static_cast<int>(n);
}
constexpr int kRouteSlicesBf16 = 4, kRouteSlicesF32 = 8;  // at most
inline int route_tile_slices(int d, int MB, int kind, bool bf16) {
  const int nch = static_cast<int>((static_cast<size_t>(d) * (bf16 ? 2 : 4) + 127) / 128);
  const int s = route_tile_smax(MB, !bf16 ? kRouteSlicesF32 : kind == 0 ? 2 : kRouteSlicesBf16);
  return s < nch ? s : nch;
}
constexpr size_t kRouteTileArea = size_t{16} << 20;   // what a workspace holds for them at least, given the tokens
constexpr size_t kRouteTileLaunch = size_t{1} << 30;  // what one launch fills of a larger area at most
// Tiles of one launch, given the bytes for its partial products: as many as fit
// them, one at least. The kernels address a launch's products by 32-bit offsets
// within 2 GiB; the area of a workspace that also serves the split-K form (1152
// bytes a token) passes that at 1.9 million tokens.
inline size_t route_tile_step(size_t bytes, int S, int MB) {
  const size_t n = (bytes < kRouteTileLaunch ? bytes : kRouteTileLaunch) / (static_cast<size_t>(S) * MB * 4096);
  return n < 1 ? 1 : n;
}
// Operands of the finishing kernel in its own layout: F as matrix-core
// fragments of whole 16 x 16 blocks, W2 in the lanes' order, padded biases.
inline size_t route_fold_floats(int Hr, int G, int C, int kind) {
  const size_t nb = route_tile_blocks(Hr, G, 0, kind), rb = route_tile_blocks(C, C, 0, 0);
  return nb * rb * 256 + (kind == 0 ? nb * G * 16 : 0) + rb * 16 + nb * 16;
}
// Bytes of folded operands and partial products, enough for kRouteTileArea of
// the latter; never falls as B or T grows (a workspace sized for a batch serves
// every smaller one). Calls with more tokens than the area holds run in several
// launches.
inline size_t route_tile_bytes(int B, int T, int Hr, int G, int C, int kind) {
  const int MB = route_tile_blocks(Hr, G, C, kind);
  const size_t tiles = (static_cast<size_t>(B) * T + 63) / 64;
  const size_t bytes = tiles * route_tile_smax(MB, kRouteSlicesF32) * MB * 4096;
  return (bytes < kRouteTileArea ? bytes : kRouteTileArea) + route_fold_floats(Hr, G, C, kind) * sizeof(float);
}
hipError_t launch_route_tile(const RouteParams& p, bool bf16, size_t part_bytes, hipStream_t s);
// Shares of the language terms (p.pcb), folded role terms (p.F) and cleared
// tile counters for the one-kernel forms, any hidden size of 16-byte rows.
void launch_pool_any(const RouteParams& p, hipStream_t s);
// Pooled language states, language terms (p.cb) and folded role terms (p.F)
// for any strides and alignment.
void launch_pool_proj(const RouteParams& p, bool bf16, hipStream_t s);

// Tokens up to which the two-kernel form is the faster one where the
// one-kernel forms apply: at d = 4096, G = 8, 48 language tokens of 177, 21.6
// against 31.8 us (1 prefix), 27 against 33.2 (16 prefixes), even at about 24
// prefixes, where its pooling blocks and tiles no longer fit the chip together;
// at d = 1024 17.4 against 28.6 (5 prefixes of 561). The line is d = 4096's, drawn
// below the crossing; at smaller d the two-kernel form is still ahead there (17
// prefixes, d = 1024: 16.7 and 22.3). Both give the same bits.
constexpr size_t kRouteTileMaxTok = 3072;
// Whether the one-kernel forms can take a call (a function of shape, type and
// alignment): bf16 MLP2 routers of 128 units whose operands are rows of whole
// 16-byte pieces from 16-byte boundaries, which is what their LDS DMA copies, and
// language terms within 2 GiB.
inline bool route_one_kernel_ok(const RouteParams& p, bool bf16) {
  const size_t ntok = static_cast<size_t>(p.B) * p.T, ncb = (static_cast<size_t>(p.d) + 511) / 512;
  return bf16 && p.kind == 0 && p.Hr == 128 && p.C >= 1 && p.C <= 16 && p.G <= 32 && p.d % 64 == 0 && p.d_e % 8 == 0 &&
         ntok < (size_t{1} << 30) && ncb * p.B * 128 * sizeof(float) < (size_t{1} << 31) &&
         ((reinterpret_cast<uintptr_t>(p.h) | reinterpret_cast<uintptr_t>(p.W1) | reinterpret_cast<uintptr_t>(p.W_r) |
           reinterpret_cast<uintptr_t>(p.E)) & 15) == 0;
}
// Whether a call with all the workspace it asks for runs in the two-kernel form.
inline bool route_uses_tiles(const RouteParams& p, bool bf16) {
  return !route_one_kernel_ok(p, bf16) || static_cast<size_t>(p.B) * p.T <= kRouteTileMaxTok;
}
hipError_t launch_route(const RouteParams& p, bool bf16, hipStream_t s);
hipError_t launch_select(const RouteParams& p, hipStream_t s);

// Role-driven within-type group allocation (and optional selection).
constexpr int kAllocMaxT = 4096;  // tokens per sample
struct AllocParams {
  int B, T, G;
  int k_by_type[4];
  const float* priority;   // [B][T]
  const uint8_t* types;    // [B][T]
  const float* scores;     // [B][T][G] or null (no selection)
  uint8_t* k_out;          // [B][T] or null
  uint32_t* mask;          // [B][T], with scores
  uint8_t* idx;            // [B][T][G] or null
  uint8_t* count;          // [B][T] or null
};
hipError_t launch_allocate(const AllocParams& p, hipStream_t s);

// Full-width routing space: one R over d_v = H*dh value dims, S groups of ds.
constexpr int kFullMaxT = 4096, kFullMaxB = 1024;
struct FullParams {
  int B, T, H, dv, S, ds;
  int64_t cap;
  const uint32_t* mask;  // [B][T]
  int32_t* offsets;      // [B][T+1]: written by the rotate step, read by the values step
  int32_t* counts;       // [B] routed tokens per sample (workspace)
  int32_t* rlist;        // [B][T] routed token indices (workspace)
  int32_t* counts_g;     // [B][S] routed tokens keeping group g (workspace)
  int32_t* starts_g;     // [B][S] start of group g's list in pairs[b] (workspace)
  int32_t* pairs;        // [B][T*S] per sample: the routed tokens keeping group 0, then 1, ... (workspace)
  const void* v;         // [B][T][dv] (rotate)
  const void* Rm;        // [dv][dv]: R^T (rotate) or R (values)
  void* Vp;              // [B][cap][ds] cache: written (rotate) or read (values)
  void* Vh;              // [B][H][T][dh] routed values (values)
};
// mode 0: rotate + pack; mode 1: values from the cache
hipError_t launch_full(const FullParams& p, int mode, hipStream_t s);
hipError_t launch_transpose(const void* R, void* Rt, int n, hipStream_t s);

struct RotateParams {
  int ntok, T, H, G, tok_per_wg;
  const void* v;
  const void* R;
  void* z;                  // rotate only
  const uint32_t* mask;     // fused rotate + pack
  int32_t* offsets;         // written by the matrix-core kernel (head 0's workgroups) unless off_ready
  int off_ready;            // offsets already hold the scan (long prefixes)
  int dyn_tiles;            // all workgroups resident at once: tiles handed out on demand
  void* Vp;
  int64_t cap;
};
hipError_t launch_rotate(bool bf16, int ntok, int H, int dh, const void* v, const void* R, void* z,
                         hipStream_t s);
// Fused rotation + pack; also writes the offsets (the exclusive scan of the
// kept counts per sample).
hipError_t launch_rotate_pack(bool bf16, int B, int T, int H, int dh, int G, const void* v, const void* R,
                              const uint32_t* mask, int32_t* offsets, void* Vp, int64_t cap,
                              hipStream_t s);
hipError_t launch_pack_offsets(int B, int T, int G, const uint32_t* mask, int32_t* offsets, hipStream_t s);

hipError_t launch_pack(bool bf16, int B, int T, int H, int dh, int G, const void* z,
                       const uint32_t* mask, int32_t* offsets, void* Vp, int64_t cap,
                       hipStream_t s);

struct AttendParams {
  int B, T, H, dh, G, Tq;
  const void *q, *k;
  const uint32_t* mask;
  const int32_t* offsets;
  const void* Vp;
  int64_t cap;
  const void* R;
  float scale;
  void* out;
  int out_f32;
  int causal;  // prefix self-attention: Tq == T and query t sees keys 0..t
  int dense;   // plain per-head values Vp = [B][H][T][dh]: no masks, offsets or rotation
};
hipError_t launch_attend(const AttendParams& p, bool bf16, hipStream_t s);

// Token retention (Sec. 3.1): per sample, per segment of consecutive tokens,
// the seg_keep highest scores. Segments are at most kRetainMaxSeg tokens.
constexpr int kRetainMaxSegments = 16, kRetainMaxSeg = 8192;
struct RetainParams {
  int B, N, K, n_seg;
  int seg_start[kRetainMaxSegments], seg_len[kRetainMaxSegments], seg_keep[kRetainMaxSegments],
      seg_out[kRetainMaxSegments];
  const float* scores;  // [B][N]
  int32_t* keep_idx;    // [B][K]
};
hipError_t launch_retain(const RetainParams& p, hipStream_t s);

struct GatherParams {
  int B, N, K;
  int64_t row_bytes;
  const int32_t* idx;  // [B][K]
  const void* src;     // [B][N][row_bytes]
  void* dst;           // [B][K][row_bytes]
};
hipError_t launch_gather_rows(const GatherParams& p, hipStream_t s);

}  // namespace rolesub
