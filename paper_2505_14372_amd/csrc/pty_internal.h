// pty_internal.h -- device-side descriptors shared by the kernels and the
// host orchestration of libpty (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>
#include <cstdint>

#include "pty.h"

namespace pty {

constexpr int kFlagBounds = 1;
constexpr int kFlagNonFinite = 2;
constexpr int kMaxReqs = 16;   // reconstructions per shared launch
constexpr int kMaxItems = 65535;   // positions per launch (one grid dimension holds them)

// Adam's per-step factors for step t >= 1: lr / (1 - b1^t) and
// 1 / sqrt(1 - b2^t), in double with b^t formed by repeated squaring, so that
// the host (host-side step count) and the device (device-side count) form
// the same values.
struct AdamFactors {
  float step_size, inv_sqrt_bc2;
};
__host__ __device__ inline double pow_int(double b, long long t) {
  double r = 1.0;
  while (t > 0) {
    if (t & 1) r *= b;
    b *= b;
    t >>= 1;
  }
  return r;
}
__host__ __device__ inline AdamFactors adam_factors(double lr, double b1, double b2, long long t) {
  const double bc1 = 1.0 - pow_int(b1, t), bc2 = 1.0 - pow_int(b2, t);
  return AdamFactors{(float)(lr / bc1), (float)(1.0 / sqrt(bc2))};
}

// One batch entry (probe position) of a launch; filled on the device.
struct Item {
  int req;          // index into the launch's request table
  int j;            // position index
  int ny, nx;       // integer window offset (top-left corner)
  float dy, dx;     // subpixel remainder of the position
  int valid;        // window inside the object
  int tile0;        // first workspace tile (modes follow)
  long long ck0;    // first checkpoint tile: slot s of mode m is tile ck0 + m + s * (n_items * M)
};

// One reconstruction taking part in a launch. Passed by value in the kernel
// arguments (a table of kMaxReqs), so no host-to-device staging is needed.
// The fields that every row and column pass reads come first: with the item pointer
// in front of a kernel's table, those of the first request share one 64-byte line.
// Spread over four lines, a pass waited for them one after the other: forward of one
// mode, 22 slices, 9 positions 418 -> 405 us at 256 x 256 and 429 -> 413 at 192 x 192. The
// next line holds the rest of what the last sums read, the one after that what makes the
// items and the noise model.
struct ReqDev {
  const float2* obj;        // [S][H][W]
  int S, M, H, W;
  int ck_every;             // checkpoint interval
  int live_k;               // >= 0: the live columns are exactly |k_x| <= live_k (no table lookup)
  const uint8_t* live;      // [N] 1 where the propagators' column u_x has a nonzero value, or null
                            // (no band limit): a propagation column pass leaves the other
                            // columns of its output unwritten, and their consumers read zeros
  const float4* prop_y;     // [S-1][N] (Hy / N^2, K_y bits, 0): H = [|k_x| <= K_y] Hy Hx, or null
  const float2* prop_x;     // [S-1][N] Hx
  const float2* prop;       // [S-1][N][N] propagators divided by N^2
  const float2* phat;       // [M][N][N] unitary probe spectrum
  float2* gobj;             // [S][H][W] or null
  int item0, n_items;
  const double* scale_dev;  // device double multiplying the adjoint's outputs (gradient of the
                            // caller's objective with respect to the loss), or null (1)
  int accumulate;           // add into gpos (chain kernels: gobj too) instead of overwriting
  int chain_final;          // the final column pass walks this request's items in kProbeSplit
                            // chains and keeps the probe-gradient sums in registers
                            // (k_col_final_chain) instead of storing h_hat (set per launch by
                            // set_chain_final); k_finish adds either
  float2* gphat;            // [M][N][N] probe-spectrum gradient (scratch) or null
  double* loss_out;         // device double or null
  const float* patterns;    // [J][N][N] or null
  float* I_out;             // [n_items][N][N] or null
  int loss;
  float eps, inv_sigma2;
  int modulus;              // far-field weight: 0 loss gradient, 1 modulus update (ePIE, LSQML)
  long long ck_base;        // first checkpoint tile of this request
  int tile_base;            // first workspace tile of this request
  int J;
  const float* positions;   // [J][2]
  const int32_t* batch_idx; // [n_items]
  float* emax;              // [n_items][S][2] window maxima of sum_m |psi_i|^2 and |O_i|^2 (ePIE) or null
  float* wsum;              // [S][H][W] scatter of sum_m |psi_i|^2 (LSQML) or null
  float* gpos;              // [n_items][2] or null
  float* gpos_dense;        // [J][2] or null
  const float2* probe;      // [M][N][N] (chain kernels: transformed by their first launch)
};

// Scale of the adjoint outputs: the launch's host factor times the request's
// device factor, read by each workgroup once.
__device__ __forceinline__ float adj_scale(const ReqDev& r, float scale) {
  return r.scale_dev ? scale * (float)(*r.scale_dev) : scale;
}

struct ReqTable {
  ReqDev r[kMaxReqs];
};
// passed by value with a few pointers and ints beside it: keep the kernel
// arguments under 4 KiB
static_assert(sizeof(ReqTable) + 256 <= 4096, "request table too large for the kernel arguments");

// Checkpoint tile of (item, mode m, stored slot s). Slot-major within a
// request, so the entry waves of one slice for the whole group are contiguous.
__device__ __forceinline__ size_t ck_tile(const Item& it, const ReqDev& r, int m, int slot) {
  return (size_t)it.ck0 + (size_t)m + (size_t)slot * ((size_t)r.n_items * (size_t)r.M);
}

// Where the forward row pass stores entry waves.
struct PsiStore {
  int mode;                 // 0: nowhere, 1: checkpoint slots, 2: segment buffer,
                            // 3: none, the input row spectrum is read from checkpoint slot i
                            //    (spectral checkpoints, written by the column passes)
  void* seg;                // segment buffer [tiles][seg_len][N][N] (checkpoint storage type)
  int seg_len, seg_slot;
  const void* src;          // FROM_REAL source (checkpoint buffer)
  int src_slot;
  int stop_after_store;     // skip the transmission and forward DFT
};

// Segment buffer slots a propagation column pass writes its output to while a
// segment of entry waves is recomputed with spectral checkpoints (seg null:
// none). Slice s goes to slot s - base of [tiles][len][N][N].
struct SegOut {
  float2* seg;
  int len, base;
};

// Where the adjoint row pass reads entry waves.
struct PsiLoad {
  int from_seg;             // 0: checkpoint slot i / ck_every, 1: segment buffer
  int spec;                 // the checkpoint slot holds the row spectrum F_x(psi_i) (float2)
  const void* seg;
  int seg_len, seg_base;    // slice i is at slot i - seg_base
};

struct LaunchCtx {
  hipStream_t stream;
  ReqTable reqs;
  int n_reqs, n_items, max_modes;
  int item_off;             // first item of this launch (chunked schedules)
  int resident;             // use the LDS-resident chain kernels
  int chain;                // use the register-tile chain kernels (pty_chain.hip)
  Item* items;
  float2* ws;               // tile workspace
  void* ck;                 // checkpoint buffer (float2, or __half2 when ck_half)
  int ck_half;
  float2* ramps;            // [n_items][2][N]
  const float2* tw;         // [N] roots of unity
  float* loss_part;         // [n_items][col blocks]
  float* pos_part;          // [tiles][col blocks][2] (tile = item tile0 + mode)
  int* flags;
  int emax;                 // the first forward records the window maxima (ePIE)
  int wsum;                 // the adjoint row pass scatters the illumination (LSQML)
  float* wscr;              // ordered reduction of the LSQML illumination sums: per-item
                            // sum_m |psi_i,m|^2 scratch [items][N][N], or null (atomics)
  float2* cscr;             // ordered object-gradient reduction: per-item contribution scratch
                            // [items][N][N] (the adjoint row pass stores, k_obj_gather adds), or
                            // null (float atomics)
  int defer;                // the adjoint row pass leaves each position's object-gradient
                            // contribution in its first mode's checkpoint slot of the slice
                            // (every slice stored in float), summed by the last launch
  unsigned col_live_blocks; // column blocks a propagation column pass runs (bit q: columns of
                            // block q; 0: all), the union over the launch's requests
  SegOut seg_out;           // recompute with spectral checkpoints: column-pass output slots
  int ck_spec;              // spectral checkpoints: the forward column passes write the row
                            // spectrum F_x(psi_i) of each stored entry wave into checkpoint
                            // slot i / ck_every (float2 storage, two-pass kernels)
};

void launch_items(const LaunchCtx& L, int N);
void launch_rows_fwd(const LaunchCtx& L, int N, int step, PsiStore st, bool from_real);
void launch_rows_adj(const LaunchCtx& L, int N, int step, PsiLoad psi, float scale);
void launch_col(const LaunchCtx& L, int N, int op, int step);
void launch_far_loss(const LaunchCtx& L, int N, int step, bool grad);
void launch_obj_gather(const LaunchCtx& L, int N, int step, int max_h, int max_w);
// Marks the requests of L whose final column pass runs as chains (unchunked
// launches with enough (column block, mode, chain) workgroups to fill the GPU).
void set_chain_final(LaunchCtx& L, int N, bool unchunked);
void launch_loss_reduce(const LaunchCtx& L, int N);
void launch_plain2d(int N, hipStream_t s, const float2* tw, const float2* src, float2* dst, int n_tiles,
                    bool inverse, float scale, bool accumulate);
void launch_fill(hipStream_t s, float* p, size_t n, float v);
void launch_step_advance(hipStream_t s, int64_t* step_dev);
int col_blocks(int N);

// Optimiser updates of one launch: one segment per variable, an element's
// update by the formulas in opt_element.
constexpr int kMaxOpt = 3 * kMaxReqs;
enum OptKind { OPT_SGD = 1, OPT_ADAM = 2 };
struct OptSeg {
  float *th, *m, *v;
  const float* g;
  long long n;              // floats
  union {
    double lr;              // SGD, and Adam with the count on the device
    AdamFactors f;          // Adam with the step's factors from the host
  };
  unsigned block0;          // first workgroup (set by the launcher)
  short kind;               // OptKind
  short wide;               // every pointer a multiple of 16 bytes (set by the launcher)
};
struct OptPar {
  double b1, b2;
  const int64_t* t_dev;     // Adam: the step is *t_dev + 1; null: see OptSeg::f
  float eps;
};
struct OptTable {
  // first workgroup * kMaxReqs + index into par of each segment, all bits set
  // past the last: side by side, read in one access
  unsigned at[kMaxOpt];
  OptSeg s[kMaxOpt];
  OptPar par[kMaxReqs];
  signed char par_of[kMaxOpt];   // the segments' indices into par
  int n_segs, n_pars;
};
static_assert(sizeof(OptTable) <= 4096 - 64, "the table is a kernel argument");
// workgroups of T threads for n elements, 4 a thread at a time
__host__ __device__ inline unsigned opt_blocks(long long n, int T) {
  const long long b = (n + 4 * T - 1) / (4 * T);
  return b > 65536 ? 65536u : (unsigned)b;
}
// Places the segments on workgroups of T threads; returns how many.
inline unsigned opt_layout(OptTable& t, int T) {
  unsigned blocks = 0;
  for (int k = t.n_segs; k < kMaxOpt; ++k) t.at[k] = ~0u;
  for (int k = 0; k < t.n_segs; ++k) {
    OptSeg& s = t.s[k];
    s.block0 = blocks;
    t.at[k] = blocks * kMaxReqs + (unsigned)t.par_of[k];
    const uintptr_t at = (uintptr_t)s.th | (uintptr_t)s.g | (s.kind == OPT_ADAM ? (uintptr_t)s.m | (uintptr_t)s.v : 0);
    s.wide = at % 16 == 0;
    blocks += opt_blocks(s.n, T);
  }
  return blocks;
}
void launch_opt(hipStream_t s, OptTable t);

enum ColOp { COL_SHIFT = 0, COL_PROP = 1, COL_PROP_ADJ = 2, COL_FINAL = 3 };

// Cost-regularizer weights on the device side (float).
struct RegDev {
  float obj_l2, obj_l1, obj_tikhonov, obj_tv, layers_tikhonov, layers_tv, tv_delta, obj_phase_l1;
};
constexpr int kMaxBlurSlices = 64;

int launch_reg_object(hipStream_t s, const float2* O, float2* g, int S, int H, int W, const RegDev& rg,
                      float* cost_part);
int launch_reg_probe(hipStream_t s, const float2* P, float2* g, size_t n, float w, float* cost_part);
// Probe phase-plate Tikhonov (wt) / TV (wv) on the unitary spectra phat [M][N][N]
// (FFT order): writes the gradient with respect to phat into gphat and cost
// partials; returns the number of partials.
// Spectral L1 step between the forward and inverse FFTs of the object slices
// (see k_spec_l1); returns the number of cost partials.
int launch_spec_l1(hipStream_t s, float2* spec, size_t n, size_t HW, float w, float* cost_part);
void launch_cadd_inplace(hipStream_t s, float2* g, const float2* a, size_t n);
int launch_reg_probe_phase(hipStream_t s, const float2* phat, float2* gphat, int M, int N, float wt, float wv,
                           float delta, float* cost_part);
void launch_add_cost(hipStream_t s, const float* part, int n, double* loss);
void launch_amp_clamp(hipStream_t s, float2* O, size_t n, float lo, float hi);
void launch_layer_blur(hipStream_t s, float2* O, int S, size_t HW, const float* g, int r);
void launch_mask_tiles(hipStream_t s, float2* t, const uint8_t* mask, size_t n, int N2);
// In-plane periodic Gaussian low pass of every slice; tmp holds S*H*W values.
void launch_lowpass(hipStream_t s, float2* O, float2* tmp, int S, int H, int W, const float* w, int r);
// Blocks per slice of the deramp sums (the partials buffer holds S * this * 4 doubles).
int deramp_blocks(int H, int W);
// Affine phase removal per slice; theta: S * 3 doubles, part: see deramp_blocks.
void launch_deramp(hipStream_t s, float2* O, int S, int H, int W, double* theta, double* part);

// LSQML (Sec. 3.3) after the adjoint chain. Transparency sum over the group's
// valid items (first n_items of items): wp[r] = sum_j tau(n_j + r) with
// tau = prod_i |O_i|^2 computed once per object pixel (tau: H * W floats);
// part holds kLsqSplit * N * N floats.
constexpr int kLsqSplit = 32;
void launch_lsq_transparency(hipStream_t s, const Item* items, int n_items, const float2* O, int S, int H,
                             int W, int N, float* tau, float* part, float* wp);
// Object step: D = -g (g the chain's object accumulator), A = prev or cur + w,
// A' = A + delta max A per slice, alpha_i from double sums (part: S *
// lsq_blocks(H * W) * 3 + S doubles of partial sums, partial maxima and
// maxima; alpha: S doubles), O -= beta alpha_i g / A', cur += w.
int lsq_blocks(size_t n);
void launch_lsq_object(hipStream_t s, float2* O, const float2* g, const float* w, float* cur, const float* prev,
                       int S, size_t HW, float delta, double gamma, float beta, double* part, double* alpha);
// Probe step, likewise with the probe accumulator g [M][N][N], the
// transparency sum wp [N][N]; alpha: 2 doubles (step, max B).
void launch_lsq_probe(hipStream_t s, float2* P, const float2* g, const float* wp, float* cur, const float* prev,
                      int M, int N2, float delta, double gamma, float beta, double* alpha);

// Is an object gradient summed strip by strip (k_object_strips), where `items`
// windows with `parts` contributions each lie on an H x W object and `slices` of it
// are summed? A workgroup per tile (object_sum) costs about 3 ns of a launch however
// little lies on its 4 x 64 values; a wave per strip less, but it adds the strip's
// contributions alone. So strips are taken where there are enough to fill the GPU,
// and few contributions over a value for their number. Over 300 calls (64, 128 and
// 256 wide windows, 1 - 6 modes, 1 and 6 slices, 8 - 512 positions on objects of 128 to
// 2000 rows) this line is within 0.3% of the better one on average; loss and
// gradients of one mode, 64 x 64, 16 positions on 2048 x 2048, tiles against strips:
// 8 slices 541 -> 179 us, one 95 -> 58; 128 positions of two modes, 6 slices, 128 x 128 on
// 800 x 800 (6.6 contributions over a value, 3900 strips), kept on tiles: 498 against 522;
// 128 half-stored positions, 6 slices summed one by one, 64 x 64 on 1536 x 1536 (2304 strips),
// kept on tiles: 396 against 431.
// A value's sum is the same bits either way.
constexpr int kStripRows = 16;
__host__ __device__ inline bool sum_in_strips(int N, long long items, int parts, int H, int W, int slices) {
  const long long strips = (long long)slices * ((H + kStripRows - 1) / kStripRows) * ((W + 63) / 64);
  const long long over = items * parts * N * N, values = (long long)H * W;   // contributions over a value: over / values
  return strips >= 3000 && over < 16 * values && over * 700 / strips < values;
}

// Last sums of the adjoint (pty_finish.hip): gather: the object gradient of slices lo ..
// lo + slices - 1 from stored contributions; rest: probe spectrum, loss, positions.
struct FinishRun {
  int lo, slices;           // slices of the object-gradient sum (0: none)
  const float2* seg;        // as in ChainRun
  int seg_len, seg_base;
  // (set by finish_layout)
  int rest, n_reqs, wide;
  unsigned strips;             // requests (bits) whose object gradient is summed in strips
  // first workgroup of each request's object-gradient tiles, and of the rest of its work,
  // which comes after the tiles of all (a tile takes longest); then that of the positions
  unsigned tiles_at[kMaxReqs], rest_at[kMaxReqs + 1];
  unsigned first;              // first workgroup of this launch
};
constexpr int kFinishTY = 4;      // rows of an object-gradient tile
// Probe pixels of a workgroup: 32, the 16 interleaved sums of each side by side, or
// (wide) 512, a thread taking the 16 of one pixel in turn: a workgroup costs about 3 ns
// of the launch, the sums in turn the latency of every fourth item. Loss and
// gradients of one slice, 32 against 512: 256 x 256, 8 modes (524288 pixels), 4
// positions 227 -> 193 us, 256 positions 2485 -> 2449; 192 x 192, 8 modes, 64 positions 491 -> 463;
// 128 x 128, 4 modes (65536), 16 positions 127 -> 126; kept at 32: the same with 64
// positions 150 against 166, 256 x 256, 2 modes, 64 positions 238 against 243. The same bits
// either way.
__host__ __device__ inline int finish_pixels(int wide) { return wide ? 512 : 32; }
inline bool finish_wide(long long pixels, long long most_items) {
  return pixels >= 262144 || (pixels >= 32768 && pixels >= 4096 * most_items);
}
// HIP takes fewer than 2^32 threads in a grid dimension: workgroups of 512 in one launch
constexpr unsigned kFinishBlocks = (1u << 23) - 1;

// Workgroups of a request: object-gradient tiles (tx x ty of each slice; none where
// the sum is taken in strips), probe pixels, loss.
struct FinishParts {
  unsigned tx, ty, gather, probe, loss;
};
__host__ __device__ inline FinishParts finish_parts(const FinishRun& p, const ReqDev& r, int q, int N) {
  FinishParts f{};
  f.tx = (unsigned)(r.W + 63) / 64;
  f.ty = (unsigned)(r.H + kFinishTY - 1) / kFinishTY;
  const int slices = r.S - p.lo < p.slices ? r.S - p.lo : p.slices;
  if (r.gobj && slices > 0 && !((p.strips >> q) & 1u)) f.gather = (unsigned)slices * f.ty * f.tx;
  if (p.rest && r.gphat) f.probe = (unsigned)r.M * (unsigned)(N * N / finish_pixels(p.wide));
  if (p.rest && r.loss_out) f.loss = 1;
  return f;
}
// Gives each request workgroups for its own sizes, and the position gradients
// theirs; returns how many there are. chain: one contribution per mode.
inline unsigned finish_layout(FinishRun& p, const ReqTable& reqs, int n_reqs, int n_items, int N, bool chain,
                              bool rest) {
  p.rest = rest ? 1 : 0;
  p.n_reqs = n_reqs;
  long long pixels = 0, most = 0;
  p.strips = 0;
  for (int q = 0; q < n_reqs; ++q) {
    const ReqDev& r = reqs.r[q];
    const int slices = r.S - p.lo < p.slices ? r.S - p.lo : p.slices;
    if (r.gobj && slices > 0 && sum_in_strips(N, r.n_items, chain ? r.M : 1, r.H, r.W, slices)) p.strips |= 1u << q;
    pixels += r.gphat ? (long long)r.M * N * N : 0;
    most = most > r.n_items ? most : r.n_items;
  }
  p.wide = finish_wide(pixels, most) ? 1 : 0;
  unsigned g = 0;
  for (int q = 0; q < kMaxReqs; ++q) {
    p.tiles_at[q] = q < n_reqs ? g : ~0u;
    if (q < n_reqs) g += finish_parts(p, reqs.r[q], q, N).gather;
  }
  for (int q = 0; q <= kMaxReqs; ++q) {
    p.rest_at[q] = q <= n_reqs ? g : ~0u;
    if (q >= n_reqs) continue;
    const FinishParts f = finish_parts(p, reqs.r[q], q, N);
    g += f.probe + f.loss;
  }
  return rest ? g + (unsigned)(n_items + 511) / 512 : g;
}
// Work of workgroup g: its request (n_reqs: the positions) and which of its tiles, or
// which of the rest.
struct FinishWork {
  bool tile;
  int req;
  unsigned index;
};
// (One request, the usual case, needs two comparisons; the search through the tables takes
// 0.3 us of a launch of 15.)
__host__ __device__ inline FinishWork finish_work(const FinishRun& p, unsigned g) {
  FinishWork w{g < p.rest_at[0], -1, 0};
  if (p.n_reqs == 1) {
    w.req = g >= p.rest_at[1] ? 1 : 0;
    w.index = w.tile ? g : g - (w.req ? p.rest_at[1] : p.rest_at[0]);
    return w;
  }
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
#endif
  for (int k = 0; k <= kMaxReqs; ++k) {
    const unsigned at = !w.tile ? p.rest_at[k] : k < kMaxReqs ? p.tiles_at[k] : ~0u;
    if (at <= g) {
      w.req = k;
      w.index = g - at;
    }
  }
  return w;
}
void launch_finish(const LaunchCtx& L, int N, FinishRun p, bool rest, float scale);

// Object gradient of one request from stored contributions, strip by strip.
struct StripRun {
  const float2* src;        // contribution `part` of item b in slice i: tile index + part * step, index:
  const float* wsrc;        // LSQML illuminations, stored alike, or null
  int scratch;              // 1: b (src is the scratch area of one slice), 0: the item's
                            // checkpoint or segment tile (as in k_finish)
  const float2* seg;
  int seg_len, seg_base;
  int parts;                // contributions of an item
  int lo, slices;           // slices lo .. lo + slices - 1
  int item_lo, item_hi;     // items of the launch
  int add;                  // add to the gradient instead of writing it
  int scaled;               // times the adjoint scale (two-pass contributions have it)
  float scale;
};
void launch_object_strips(hipStream_t s, int N, const Item* items, const ReqDev& r, StripRun p);

// Chain kernels (pty_chain.hip): every slice of a tile in one launch.
enum { kForward = 1, kRecompute = 2, kFar = 4, kSeed = 8, kAdjoint = 16, kFirst = 32 };   // see k_chain
struct ChainRun {
  int what;
  int store;                // kForward: store the entry waves in the checkpoint slots
  int from, to;             // kRecompute
  int hi, lo;               // kAdjoint: slices hi .. lo (hi unused with kFirst; lo -1: down to slice 0)
  float2* seg;              // entry waves of slices that are no multiples of ck_every, or null:
  int seg_len, seg_base;    // slice i at slot i - seg_base of [tiles][seg_len][N][N]
};
bool chain_size(int N);
// Items of one launch of T threads a tile, eights of them times the most modes of
// any request: HIP takes fewer than 2^32 threads in a grid dimension.
inline int chain_items(int max_modes, int T) {
  const long long n = ((1ll << 32) - 1) / T / max_modes / 8 * 8;
  return n < 8 ? 8 : n > kMaxItems + 1 ? kMaxItems + 1 : (int)n;
}
void launch_chain_begin(const LaunchCtx& L, int N);
void launch_chain(const LaunchCtx& L, int N, const ChainRun& p);
// dst[k] = scale F^-1(src[k]) (+ dst[k] if accumulate) of the n[k] N x N tiles of each entry
struct PlainTable {
  const float2* src[kMaxReqs];
  float2* dst[kMaxReqs];
  int n[kMaxReqs];
  int count;
};
void launch_chain_plain_inv(int N, hipStream_t s, const float2* tw, const PlainTable& t, float scale, bool acc);

// LDS-resident forward / adjoint chains (N = 64, 128; every slice checkpointed)
bool resident_supported(int N);
void launch_res_fwd(const LaunchCtx& L, int N, bool save);
void launch_res_adj(const LaunchCtx& L, int N, float scale);

}  // namespace pty
