// Launch arguments shared by the C-ABI layer (videomla_api.cpp) and the kernel files.
// Host-visible plain structs only; no device code here.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vmla {

constexpr int kMaxRopePairs = 64;  // a whole dense head of 128 channels
constexpr int kMaxWriteDModel = 2048;  // cache write: 32 resident x rows of d_model fill 128 KB of LDS
constexpr int kMaxWriteOutPlain = 288;   // d_c + d_rope of the plain-weight cache write
constexpr int kMaxWriteOutPacked = 576;  // d_c + d_rope of the packed-weight cache write
// 16-row output blocks per wave of the packed-weight cache write: 2 (32 outputs) up to 288
// outputs, else 4 (64 outputs), so that at most 9 waves cover d_c + d_rope
__host__ __device__ inline int write_blocks_per_wave(int outputs) { return outputs <= kMaxWriteOutPlain ? 2 : 4; }

// Per RoPE pair p (interleaved channels 2p, 2p+1 of the d_rope vector): the axis whose
// coordinate drives it (0 = t, 1 = h, 2 = w) and theta = base^(-2k / D_axis), in double.
struct RopeTable {
  int32_t n_pairs;
  int32_t axis[kMaxRopePairs];
  double theta[kMaxRopePairs];
};

struct Geometry {
  int32_t grid_h, grid_w, window_frames;
  int32_t chunk_tokens;   // chunk_frames * HW
  // Queries of an attention call: chunk tokens q_begin .. q_begin + q_count - 1 (the whole
  // chunk unless the call asks for a block of its query rows); q_count tokens per batch element
  // in the query, output and workspace tensors.
  int32_t q_begin, q_count;
  int64_t frame_end;      // absolute first frame of the chunk
  int64_t ring_tokens;    // window_frames * HW (ring rows per batch element)
  // Attention sink: frames 0 .. sink_frames-1 keep frame slots 0 .. sink_frames-1, later frames
  // cycle through the other window_frames - sink_frames slots. With a sink, positional keys are
  // cached unrotated and the context is rotated at window-local time: frame f < sink_frames at
  // f, a recent frame f at sink_frames + (f - local_lo).
  int32_t sink_frames;
  int64_t local_lo;       // first recent frame of the chunk's context (sink_frames > 0 only)
};

#ifdef VMLA_PHASE_STAMPS
// Phase stamps, in the diagnostic build only (the same sources compiled with
// VMLA_PHASE_STAMPS into libvideomla_stamps.so). Lane 0 of every wave of the stamped kernels
// writes the 100 MHz real-time counter at named points of the kernel into a caller-owned
// device buffer of uint64 [kernel][workgroup][wave][point]; the launch arguments carry the
// buffer that videomla_stamps_attach last set. The product build has neither the field nor
// the stores.
constexpr int kStampKernels = 5, kStampWorkgroups = 2048, kStampWaves = 8, kStampPoints = 16;
constexpr int64_t kStampBufferBytes =
    (int64_t)kStampKernels * kStampWorkgroups * kStampWaves * kStampPoints * 8;
enum StampKernel {
  kStampWritePacked = 0,  // cache_write_packed_kernel
  kStampWriteWide = 1,    // cache_write_wide_kernel
  kStampQAbsorb = 2,      // q_absorb_kernel
  kStampAttend = 3,       // latent_attend_kernel (latent form)
  kStampOutProj = 4,      // out_proj_kernel
};
uint64_t* stamp_buffer();  // the attached buffer, or nullptr (videomla_api.cpp)
#endif

struct WriteArgs {
#ifdef VMLA_PHASE_STAMPS
  uint64_t* stamps = stamp_buffer();
#endif
  const uint16_t* x;      // [B][chunk_tokens][d_model]
  const uint16_t* w_dkv;  // [d_c][d_model]
  const uint16_t* w_kr;   // [d_rope][d_model]
  const uint16_t* gamma;  // [d_c] or nullptr
  uint16_t* c_kv;         // [B][ring_tokens][d_c]
  uint16_t* k_r;          // [B][ring_tokens][d_rope]
  int32_t* slots;         // [chunk_tokens] or nullptr
  const uint16_t* w_packed;  // packed [W_DKV; W_KR] panel (cache_write_packed_kernel), or nullptr
  uint16_t* w_packed_out;    // pack_write_weights_kernel output
  int32_t batch, d_model, d_c, d_rope;
  int32_t tok_per_wg;     // tokens of the flat [B][chunk] order per workgroup (1 .. 32)
  int32_t n_cu;           // compute units of the device (the batched write's grid)
  float eps;
  Geometry geo;
  RopeTable rope;
};

struct AttendArgs {
#ifdef VMLA_PHASE_STAMPS
  uint64_t* stamps = stamp_buffer();
#endif
  const uint16_t* q_nope;  // [B][Nq][H][d_nope]
  const uint16_t* q_r;     // [B][Nq][H][d_rope]
  const uint16_t* w_uk;    // [H*d_nope][d_c]
  const uint16_t* w_uv;    // [H*d_v][d_c]
  const uint16_t* c_kv;    // ring
  const uint16_t* k_r;     // ring
  uint16_t* out;           // [B][Nq][H][d_v]
  uint16_t* qcat;          // workspace: [B*Nq*H][dqk_pad] bf16
  float* o_part;           // workspace: [max_seg][B*Nq*H][d_c] fp32
  float* ml_part;          // workspace: [max_seg][B*Nq*H][2] fp32 (running max, sum)
  uint16_t* k_rot;         // workspace (sink only): [B][ring_tokens][d_rope], rotated window keys
  int32_t batch, n_heads, d_nope, d_rope, d_c, d_v, dqk_pad;
  int32_t n_valid;         // valid ring slots (prefix of the ring)
  // Work partition of the attention kernel: units are (batch, row block, key tile) triples in
  // that order; workgroup w processes units [w*U/G, (w+1)*U/G). A row block whose tiles are
  // spread over k workgroups leaves k partial results, in slots 0..k-1.
  int32_t n_wg;            // G
  int32_t att_rows;        // query rows per row block
  int32_t row_blocks;      // row blocks per batch element
  int32_t tiles_per_row;   // T = ceil(n_valid / keys per tile)
  int64_t units;           // U = batch * row_blocks * T
  int32_t small_units;     // U * G < 2^32: the attention kernel's split in 32-bit arithmetic
  int32_t max_seg;         // partial-result slots the workspace holds
  float qscale;            // softmax scale * log2(e), folded into the absorbed query
  // Weighted partition (optional): the state area of kBalSlot words in the workspace (see bal_*
  // below). bal_on: split by the weights the state holds (equal weights, i.e. the even split, if
  // it holds no valid record for this G); bal_rec: the call is adaptive, bal_prep_kernel has
  // set the weights from the previous adaptive call's times and the attention kernel records
  // its own. bal_on = 0: the even split above, the state is not read.
  uint32_t* bal_state;
  int32_t bal_on, bal_rec;
  Geometry geo;
  RopeTable rope;
  // dense per-head comparator only (rows are (head, token) pairs, each head padded to nq_pad)
  const uint16_t* q;       // [B][Nq][H][d_v] unrotated queries
  const uint16_t* kv;      // ring [B][ring_tokens][H][2 * d_v]: rotated K_h, then V_h
  int32_t nq_pad;          // query rows per head, a whole number of row blocks
};

// Dense comparator's cache write: K = W_K x (rotated by 3D RoPE over each whole head), V = W_V x.
struct DenseWriteArgs {
  const uint16_t* x;       // [B][chunk_tokens][d_model]
  const uint16_t* w_k;     // [H*d_v][d_model]
  const uint16_t* w_v;     // [H*d_v][d_model]
  uint16_t* kv;            // [B][ring_tokens][H][2 * d_v]
  int32_t* slots;          // [chunk_tokens] or nullptr
  int32_t batch, d_model, n_heads, d_head;
  int32_t n_cu;            // compute units of the device
  Geometry geo;
  RopeTable rope;          // d_head / 2 pairs
};

// Plain bf16 GEMM out^T[o][token] = a[o][:] . b[token][:] (a [N][K], b [M][K], K % 64 == 0).
constexpr int kEpiStore = 0;  // out[token][o] (row stride ldo), bf16
constexpr int kEpiQcat = 1;   // q_cat rows (token, head): RMSNorm factor, RoPE, scale; see k_layer.hip
constexpr int kEpiHeads = 2;  // out[token][(o / head_w) head_ld + col_off + o % head_w], bf16, head_w % 8 == 0
struct GemmArgs {
  const uint16_t* a;       // [N][K] weight rows
  const uint16_t* b;       // [M][K] token rows
  uint16_t* out;
  int32_t M, N, K, ldo;
  int32_t epi;
  // q_cat epilogue: output column o = h (q_dc + q_dr) + c; row (token, h) of width ldo
  int32_t q_heads, q_dc, q_dr, q_norm_dim;
  // per-head epilogue: output column o goes to head o / head_w, column col_off + o % head_w
  int32_t head_w, head_ld, col_off;
  float qscale, eps;
  Geometry geo;            // token t of the flat [B][q_count] order is query t % q_count
  RopeTable rope;
};

// Packing of the whole layer's weights (see k_layer.hip).
struct PrepArgs {
  const uint16_t *w_dq, *gamma_q, *w_uq, *w_qr, *w_uk, *w_uv, *w_o;
  uint16_t *w_dq_pad, *wq_cat, *b_o;
  int32_t n_heads, d_model, d_nope, d_rope, d_c, d_v, d_q, d_q_pad, k_out_pad;
};

// floor(n / d) for n >= 0, d >= 1, exactly, without the integer division's chain of about 150
// instructions. Below 2^53 both operands are exact doubles, and the truncated, correctly rounded
// quotient is already floor(n / d): a quotient q + r/d with r >= 1 sits at least 1/d above q and
// 1/d below q + 1, more than half an ulp of it (at most n 2^-53 / d). The two correction steps only
// guard against a division that is not correctly rounded.
__host__ __device__ inline int64_t floor_div(int64_t n, int64_t d) {
  if (n >= (int64_t(1) << 53)) return n / d;
  int64_t q = (int64_t)((double)n / (double)d);
  if (q * d > n) --q;
  else if ((q + 1) * d <= n) ++q;
  return q;
}

// Workgroup whose unit range [w*U/G, (w+1)*U/G) contains `unit`.
__host__ __device__ inline int attend_owner(int64_t unit, int64_t units, int n_wg) {
  return (int)floor_div((unit + 1) * (int64_t)n_wg - 1, units);
}

// The most workgroups that share one of N row blocks of T units each, split evenly over G <= N T:
// the largest attend_owner(r T + T - 1) - attend_owner(r T) + 1. With U = N T, the owner of a row
// block's last unit is floor(((r + 1) G - 1) / N), and that of its first, with r G = a N + b, is a,
// or a + 1 where b T + G - 1 reaches U; a and b advance without a division, and the pattern repeats
// after N / gcd(N, G) row blocks. (Every call needs this for each number of frames a window can
// hold, before its first launch: 40 us at the Wan shape with two 64-bit divisions per row block.)
__host__ inline int partition_max_seg(int64_t N, int64_t T, int64_t G) {
  int64_t x = N, y = G;
  while (y) {
    const int64_t z = x % y;
    x = y;
    y = z;
  }
  const int64_t period = N / x, step_a = G / N, step_b = G % N, wrap = N * T - (G - 1);
  int64_t a = 0, b = 0, most = 1;
  for (int64_t r = 0; r < period; ++r) {
    const int64_t first = a + (b * T >= wrap);
    a += step_a;
    b += step_b;
    if (b >= N) {
      b -= N;
      ++a;
    }
    const int64_t last = b == 0 ? a - 1 : a;
    if (last - first + 1 > most) most = last - first + 1;
  }
  return (int)most;
}

constexpr int kMaxSplitsPerRowBlock = 64;
// Work partition of the attention kernel for a window of n_valid keys (see AttendArgs).
struct Partition {
  int G, rows, RB, T, max_seg;
  int64_t U;
};

// rows: query rows per row block; RB: row blocks per batch element; bn: keys per tile;
// default_wgs: workgroups resident on the device; n_wg: requested workgroups (0 = default_wgs).
__host__ inline Partition make_partition(int rows, int RB, int bn, int default_wgs, int32_t batch,
                                         int64_t n_valid, int n_wg) {
  Partition p{};
  p.rows = rows;
  p.RB = RB;
  p.T = (int)((n_valid + bn - 1) / bn);
  p.U = (int64_t)batch * p.RB * p.T;
  // by default at most kMaxSplitsPerRowBlock - 1 workgroups per row block: few-query calls
  // (few row blocks, each split over many workgroups) then give each workgroup at least 1/63 of
  // a row block's key tiles, which bounds the partial results they write, and the merge reads,
  // relative to the keys they read
  int64_t G = n_wg > 0 ? n_wg : default_wgs;
  if (n_wg == 0 && G > (int64_t)(kMaxSplitsPerRowBlock - 1) * batch * RB)
    G = (int64_t)(kMaxSplitsPerRowBlock - 1) * batch * RB;
  p.G = (int)(G < p.U ? G : p.U);
  p.max_seg = partition_max_seg((int64_t)batch * RB, p.T, p.G);
  return p;
}

// Weighted partition of the attention units. Workgroup k runs on XCD k mod 8 and gets a share of
// the units proportional to its XCD's integer weight w[k mod 8] in [kBalMin, kBalMax]:
// workgroup k takes [start(k), start(k+1)) with start(k) = floor(U cum(k) / cum(G)), cum(k) the
// summed weights of workgroups 0 .. k-1. Equal weights give the even split. The state area holds
// the weights (words 0..7), the G they were set for (8), a marker (9) and each workgroup's
// duration in 100 MHz ticks (kBalHead + k) as the last adaptive call recorded it. An adaptive
// call first runs bal_prep_kernel (one workgroup, stream-ordered between the previous call's
// last reader of the weights and this call's attention kernel): it sets each XCD's weight
// proportional to the work per time that XCD achieved, writes G and the marker, and clears the
// durations. Any state that fails the checks means equal weights.
constexpr uint32_t kBalMin = 820, kBalMax = 1280, kBalOne = 1024, kBalMark = 0x564d4c42u;
constexpr int kBalHead = 16, kBalMaxWg = 4096, kBalSlot = kBalHead + kBalMaxWg;

// The weights a partition state holds for G workgroups: its words 0..7 if the marker, G and
// every weight check out, else equal weights.
__host__ __device__ inline void bal_weights(const uint32_t* st, int G, uint32_t (&w)[8]) {
  bool ok = st[9] == kBalMark && st[8] == (uint32_t)G;
  for (int x = 0; x < 8; ++x) ok = ok && st[x] >= kBalMin && st[x] <= kBalMax;
  for (int x = 0; x < 8; ++x) w[x] = ok ? st[x] : kBalOne;
}

__host__ __device__ inline int64_t bal_cum(const uint32_t* w, int k) {
  int64_t s = 0;
  for (int x = 0; x < 8; ++x) s += (int64_t)w[x] * (k > x ? (k - x + 7) / 8 : 0);
  return s;
}
// start(k); cum_g = cum(G)
__host__ __device__ inline int64_t bal_start_at(const uint32_t* w, int64_t cum_g, int64_t U, int k) {
  return floor_div(U * bal_cum(w, k), cum_g);
}
__host__ __device__ inline int64_t bal_start(const uint32_t* w, int G, int64_t U, int k) {
  return bal_start_at(w, bal_cum(w, G), U, k);
}
// The workgroup whose range contains `unit`: the largest k < G with start(k) <= unit, i.e.
// with cum(k) <= C = floor(((unit + 1) cum(G) - 1) / U); cum(8q + j) = q S + w[0] + .. + w[j-1]
// with S the sum of the 8 weights, so k = 8 (C / S) + the number of leading weights whose sum
// stays within C mod S.
__host__ __device__ inline int bal_owner(const uint32_t* w, int G, int64_t U, int64_t unit) {
  // C <= cum(G) <= kBalMax G < 2^32 for the at most 2^20 workgroups of a call; S < 2^14
  const uint32_t C = (uint32_t)floor_div((unit + 1) * bal_cum(w, G) - 1, U);
  uint32_t S = 0;
  for (int x = 0; x < 8; ++x) S += w[x];
  int64_t r = C % S, k = (int64_t)(C / S) * 8;
  for (int x = 0; x < 7 && r >= (int64_t)w[x]; ++x) {
    r -= w[x];
    ++k;
  }
  return (int)(k < G - 1 ? k : G - 1);
}

// Partial-result slots a row block of T units can need under any weights: every range holds at
// least floor(U kBalMin / (kBalMin + (G - 1) kBalMax)) - 1 units. More than any workspace has
// (kBalNever) where that is none: a range could be empty.
constexpr int kBalNever = 0x7fffffff;
__host__ __device__ inline int bal_max_seg(int G, int64_t U, int T) {
  const int64_t min_len = U * kBalMin / (kBalMin + (int64_t)(G - 1) * kBalMax) - 1;
  if (min_len < 1) return kBalNever;
  const int64_t n = (T + min_len - 1) / min_len + 1;
  return (int)(n < G ? n : G);
}
// Whether a call may take the weighted split: every range keeps at least one unit under any
// weights (the merges count the owners between a row block's first and last, each of which must
// have written its partial result), and the workspace's n_seg partial-result slots hold what such
// ranges can leave. n_seg is the most that any window of the shape needs, so a window that is
// still filling, with fewer units, must not be admitted for its number of slots alone.
__host__ inline bool weighted_split_fits(const Partition& p, int n_seg) {
  const int need = bal_max_seg(p.G, p.U, p.T);
  return p.G <= kBalMaxWg && need != kBalNever && need <= n_seg;
}

// Whether the dense cache write takes its 256 x 256 tiles instead of the 128 x 128 ones. Rounds of
// one workgroup per compute unit: a round of wide tiles (four times the work) takes about as long
// as two of the small ones: 40 to 54 us a round, the fuller the longer, against 25 for one and 20
// for each further one at d_model = 1536, 27 to 32 against 18 and 13 at 768 (2 against 1 rounds:
// 40.2 against 45.2 us at 1,560 tokens x 12 heads, 4 against 1: 83.6 against 52.3 at 3,120 x 16).
// d_head % 8: the wide kernel's stores, 16-byte chunks, stay inside a head.
constexpr int kDenseTile = 128, kDenseWideTile = 256;
__host__ inline int64_t dense_wide_tiles(int64_t M, int64_t N) {
  return (M + kDenseWideTile - 1) / kDenseWideTile * ((N + kDenseWideTile - 1) / kDenseWideTile);
}
__host__ inline bool dense_write_wide(int64_t batch, int64_t tokens, int64_t n_heads, int64_t d_head,
                                      int64_t n_cu) {
  const int64_t M = batch * tokens, N = 2 * n_heads * d_head, wide = dense_wide_tiles(M, N);
  const int64_t small = batch * ((tokens + kDenseTile - 1) / kDenseTile) * (N / kDenseTile);
  auto rounds = [&](int64_t tiles) { return (tiles + n_cu - 1) / n_cu; };
  return d_head % 8 == 0 && rounds(small) > 2 * rounds(wide) && M + kDenseWideTile < (1LL << 31) &&
         wide < (1LL << 31);
}

// Whether the partial results of a call of `rows` query rows, each split over up to `splits`
// workgroups, are merged by a workgroup per row (vmla_merge.h) instead of a thread per 8 columns.
// While the bytes are few, the first takes about 4 us and 2.5 us per 1,000 rows, whatever the splits;
// the second waits for its loads in turn, 3 us and 0.2 us per split in the latent merge (groups of
// four in flight), 2 us and 0.5 us per split in the per-head one (one at a time beyond four). us,
// workgroup / thread:
//   latent, rows x splits   192 x 7    768 x 12   1536 x 12   1536 x 32   2400 x 20   3840 x 63
//     d_c = 64              4.5 / 4.0  5.1 / 6.1  6.7 / 5.4   8.5 / 10.9  10.8 / 8.5  16.3 / 17.9
//     d_c = 192             4.9 / 4.7  5.2 / 6.0  7.9 / 6.5  10.0 / 11.0  11.3 / 9.5  31.1 / 31.3
//     d_c = 512             4.8 / 4.7  6.8 / 7.1  9.6 / 8.9  16.8 / 18.1  17.2 / 18.3  129 / 132
//   per head, 128 columns   768 x 5    1536 x 5   1536 x 12   3840 x 12   3840 x 32   12288 x 63
//                           4.0 / 4.7  5.8 / 4.8  6.4 / 8.2  12.6 / 9.5  15.0 / 21.1  96 / 107
// Over 390 such points (rows 12 to 12,288, splits 5 to 63, every width) the rule is at most 7% slower
// than the better of the two; wider rows than 192 columns differ by 7% at most beyond its line (both
// are then bound by the bytes), so the width is left out.
__host__ inline bool merge_by_workgroup(int64_t rows, int splits, bool per_head) {
  const int64_t least = per_head ? 4 : 8, per_split = per_head ? 200 : 75;
  return splits > least && rows <= per_split * splits && rows < (1 << 24);  // (one grid)
}

// Sets the calling thread's last-error message (videomla_last_error) and returns `code`; for
// the C-ABI sources other than videomla_api.cpp.
int report_error(int code, const char* fmt, ...);

// Launchers (one per kernel). Return the launch status.
hipError_t launch_cache_write(const WriteArgs& a, hipStream_t s);
int cache_write_tokens_per_wg(int64_t tokens, int n_cu);
hipError_t launch_pack_write_weights(const WriteArgs& a, hipStream_t s);
size_t write_weights_packed_elems(int d_model, int d_c, int d_rope);
hipError_t launch_q_absorb(const AttendArgs& a, hipStream_t s);
hipError_t launch_rope_window(const AttendArgs& a, hipStream_t s);
hipError_t launch_bal_prep(const AttendArgs& a, hipStream_t s);
hipError_t launch_latent_attend(const AttendArgs& a, hipStream_t s);
hipError_t launch_latent_attend_wide(const AttendArgs& a, hipStream_t s);  // d_c = 512
constexpr int kWideRows = 64, kWideKeys = 32;  // its row block and key tile
// out_proj of a call whose row blocks can be split over more workgroups than its in-kernel
// merge table holds (few-query calls): launch_latent_merge first writes the merged bf16 o_lat rows
// [row][d_c] into the q_cat area (ld_olat = n_heads * d_c), which out_proj then reads.
bool out_proj_premerged(const AttendArgs& a);
hipError_t launch_out_proj(const AttendArgs& a, hipStream_t s);
hipError_t launch_dense_cache_write(const DenseWriteArgs& a, hipStream_t s);
hipError_t launch_dense_q_prep(const AttendArgs& a, hipStream_t s);
hipError_t launch_dense_attend(const AttendArgs& a, hipStream_t s);
hipError_t launch_dense_merge(const AttendArgs& a, hipStream_t s);
hipError_t launch_mat_q_prep(const AttendArgs& a, hipStream_t s);
hipError_t launch_mat_attend(const AttendArgs& a, hipStream_t s);
bool mat_attend_supported(int d_k, int d_v);
hipError_t launch_mat_rope_fill(const AttendArgs& a, uint16_t* kv, hipStream_t s);
hipError_t launch_gemm_nt(const GemmArgs& a, hipStream_t s);
hipError_t launch_latent_merge(const AttendArgs& a, uint16_t* o_lat, int ld_olat, hipStream_t s);
hipError_t launch_prepare_weights(const PrepArgs& a, hipStream_t s);

// Shapes the attention kernel is instantiated for.
bool latent_attend_supported(int d_c, int d_rope);
size_t q_absorb_lds_bytes(int d_c, int d_rope, int d_nope);
int latent_attend_rows_per_block(int d_c, int d_rope);
int latent_attend_keys_per_tile(int d_c, int d_rope);
int latent_attend_wgs_per_cu(int d_c, int d_rope);
bool dense_attend_supported(int d_head);
int dense_attend_rows_per_block();
int dense_attend_keys_per_tile();

}  // namespace vmla
