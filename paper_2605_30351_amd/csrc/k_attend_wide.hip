// latent_attend for wide latents (d_c = 512): the same product as latent_attend_kernel
// (k_attend.hip), S^T = [c_kv | k_r] q_cat^T, online softmax in base 2, O_lat^T += c_kv^T P^T over
// one key range, with the work of a 64-row block split over four waves.
//
// What bounds it: a row's fp32 accumulators (512 columns) leave room for 64 rows per compute unit
// at one wave per SIMD, and every 32-key tile is read from LDS for those 64 rows only. A 32x32x16
// MFMA whose A operand is read for 32 rows takes 1 KB of LDS per 32 cycles and SIMD, half of what
// LDS delivers (256 B per cycle, in 16-byte and in transposed reads alike, measured), and the one
// wave of a SIMD has nothing to run while it waits; so the split is chosen for the fewest LDS bytes:
//   scores   wave (r, k) takes the rows 32 r .. +32 and the keys 16 k .. +16 of the tile, over all
//            columns (MFMA 16x16x32, the K operand shared by two 16-row blocks): 17 KB;
//   P^T      goes through LDS as bf16 (4 KB per tile), so that every score is computed and
//            exponentiated once;
//   PV       wave w takes the columns 128 w .. +128 of all 64 rows (MFMA 32x32x16, the V operand
//            shared by two 32-row blocks): 8 KB, and 4 KB of P^T.
// 30 KB per wave and tile. The version before (pairs of waves that each contracted half of the
// columns for 32 rows, exchanged fp32 partial scores and both exponentiated them) read and wrote
// 41 KB. Wan chunk of 4,680 tokens x 12 heads over 32,760 keys, whole attend: 4720 us before, 3500
// now (1.11 PFLOP/s). The matrix pipes are busy 48% of the cycles at 2.0 GHz; what is left is the
// 35 KB of tile that every compute unit takes in per 64 rows (without these loads: 3050 us).
//
// A step t runs the score MFMAs of tile t+1 with the softmax of tile t under them, a barrier that
// publishes P(t), then the PV MFMAs of tile t with the row max of tile t+1 under them, and a
// barrier that publishes that max. A ring of four tiles: tile t+3 is loaded from global memory
// during step t and first read (the first score operands) at the end of step t+1.
//
// Tile layout: c_kv [32][512], row-major, 16-byte chunk c of row r at c XOR (4 (r mod 4) + h(r)),
// h(r) = -(r / 4) mod 4; then k_r [32][32], chunk c at c XOR h(r). One load instruction fills one
// c_kv row, so that its address is scalar. A 16-byte LDS read serves the lanes {0-3, 12-15, 20-27},
// {4-11, 16-19, 28-31} (and these + 32) together: in the score operand reads (row l mod 16, chunk
// 4 ks + l / 16) these lanes see h = 0, 3, 1 ^ h(4), 1 ^ h(8), all different, and with the row's
// 4 (r mod 4) hit 16 different bank groups; h(r) = (r / 4) mod 4 gave two lanes per group
// (conflicts in 37% of the LDS cycles, now 6%). The 4-row transpose reads of the PV MFMA hit 16
// different groups with either.
#include "vmla_device.h"

namespace vmla {
namespace {

constexpr float kNegInfW = -__builtin_huge_valf();
constexpr float kLazyMaxW = 8.0f;  // the running max is raised by more than this only (log2 units)

// D(16x16) += A(16x32) B(32x16). Lane l holds A[l%16][8(l/16) .. +8], B[8(l/16) .. +8][l%16];
// accumulator element i of lane l is D[4(l/16) + i][l%16].
__device__ __forceinline__ f32x4 mfma16w(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// s_waitcnt with only the LDS counter constrained (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  static_assert(N >= 0 && N < 16, "lgkmcnt range");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (N << 8));
}

// Workgroup barrier alone: the callers wait for the LDS operations that it publishes, so that
// operand reads issued after those stay in flight across it.
__device__ __forceinline__ void bare_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Largest / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ __forceinline__ float quad_max(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return half_swap_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quad_sum(float v) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return half_swap_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

struct WideCfg {
  static constexpr int DC = 512, DR = 32;
  static constexpr int NW = 4, ROWS = kWideRows, BN = kWideKeys, NBUF = 4;
  static constexpr int DQK = DC + DR;
  static constexpr int KS = DQK / 32;            // score steps of 32 columns
  static constexpr int DB = DC / 32 / NW;        // 32-column value blocks per wave
  static constexpr int TILE = BN * DQK;          // elements
  static constexpr int CL = BN / NW;             // c_kv rows (loads) per wave and tile
  static constexpr int RL = BN * DR / 512;       // k_r loads per tile, by waves 0 .. RL-1
  static_assert(RL <= NW && CL == 2 * DB, "one load per c_kv row and value slot");
  // chunk c of row r sits at c ^ swz(r) (k_r rows, of four chunks: c ^ swz4(r))
  static constexpr int swz4(int r) { return -(r >> 2) & 3; }
  static constexpr int swz(int r) { return ((r & 3) << 2) | swz4(r); }
};

__global__ __launch_bounds__(256, 1) void latent_attend_wide_kernel(const AttendArgs a) {
  using C = WideCfg;
  constexpr int DC = C::DC, DR = C::DR, BN = C::BN, DB = C::DB, KS = C::KS;
  __shared__ __attribute__((aligned(16))) uint16_t tile[C::NBUF][C::TILE];
  __shared__ __attribute__((aligned(16))) uint16_t pbuf[2][2][2][32][8];  // [rows/32][kk][g][row][key]
  __shared__ float mx[2][C::ROWS];                                       // [key half][row]
  __shared__ __attribute__((aligned(16))) float resc[C::NW][64 * 16];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, l32 = lane & 31;
  const int qd = lane >> 4, l16 = lane & 15;
  const int rh = wave & 1, kh = wave >> 1;  // score rows 32 rh .., keys 16 kh ..
  const int rows_b = a.geo.q_count * a.n_heads;
  VMLA_STAMP(a, kStampAttend, 0);
  int stamp_step = 0, stamp_seg = 0;  // steps taken, segments finished (phase stamps only)

  // this workgroup's share of the (batch, row block, key tile) units, as in latent_attend_kernel
  const int64_t U = a.units;
  const int G = a.n_wg, T = a.tiles_per_row;
  auto uniform = [](int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
  };
  int64_t u_begin, u_end;
  uint32_t bw[8];
  uint64_t bal_t0 = 0;
  if (a.bal_on) {
    bal_weights(a.bal_state, G, bw);
#pragma unroll
    for (int x = 0; x < 8; ++x) bw[x] = __builtin_amdgcn_readfirstlane(bw[x]);
    const int64_t cum = bal_cum(bw, G);
    u_begin = uniform(bal_start_at(bw, cum, U, blockIdx.x));
    u_end = uniform(bal_start_at(bw, cum, U, blockIdx.x + 1));
    if (a.bal_rec) bal_t0 = __builtin_amdgcn_s_memrealtime();
  } else {
    u_begin = uniform(floor_div((int64_t)blockIdx.x * U, G));
    u_end = uniform(floor_div((int64_t)(blockIdx.x + 1) * U, G));
  }
  // Segments (runs of tiles of one row block) in this order: whole row blocks first, then the
  // head of one (keys from 0), then the tail of one. Every whole block and the heads start at key
  // 0, so that all workgroups walk the keys at about the same position at the same time and those
  // of one XCD find most tiles in its L2.
  const int64_t rb_lo = uniform(floor_div(u_begin, T)), rb_hi = uniform(floor_div(u_end - 1, T));
  const int n_seg = (int)(rb_hi - rb_lo) + 1;
  const int head = n_seg > 1 && u_end < (rb_hi + 1) * T, tail = n_seg > 1 && u_begin > rb_lo * T;

  // loads: c_kv row wave + 4 i of a tile (lane l fetches the chunk whose place is l), at byte
  // offset coff[i] from the tile's first row; k_r rows 16 wave .. +16 (waves 0 and 1)
  uint32_t coff[C::CL];
#pragma unroll
  for (int i = 0; i < C::CL; ++i)
    coff[i] = (uint32_t)((wave + 4 * i) * DC * 2 + (lane ^ C::swz(wave + 4 * i)) * 16);
  const int krow = 16 * wave + (lane >> 2), kch = (lane & 3) ^ C::swz4(krow);

  // LDS element offsets inside a tile. Scores: row 16 kh + l16, chunk 4 ks + qd, whose XOR
  // leaves ks / 4 alone: one base per ks mod 4. PV: rows 4 g + tr_row (+ 8) of a 16-key block,
  // columns tr_col of the wave's value block d (see lds_read_tr).
  int kofs[4], vlo[DB], vhi[DB];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    kofs[i] = (16 * kh + l16) * DC + ((4 * i + qd) ^ C::swz(l16)) * 8;
  const int kofs_r = BN * DC + (16 * kh + l16) * DR + (qd ^ C::swz4(l16)) * 8;
  const int tr_row = (lane & 15) >> 2;
  const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    const int ch = (wave * DB + d) * 4 + (tr_col >> 3);
    vlo[d] = (4 * g + tr_row) * DC + (ch ^ C::swz(4 * g + tr_row)) * 8 + (tr_col & 7);
    vhi[d] = (4 * g + tr_row + 8) * DC + (ch ^ C::swz(4 * g + tr_row + 8)) * 8 + (tr_col & 7);
  }

  for (int seg = 0; seg < n_seg; ++seg) {
    const int64_t rbg = seg < n_seg - head - tail ? rb_hi - head - seg
                        : head && seg == n_seg - head - tail ? rb_hi : rb_lo;
    const int b = (int)uniform(floor_div(rbg, a.row_blocks));
    const int rb = (int)(rbg - (int64_t)b * a.row_blocks);
    const int kt0 = (int)(max(u_begin, rbg * T) - rbg * T);
    const int n_tiles = (int)(min(u_end, (rbg + 1) * T) - rbg * T) - kt0;
    int split = 0;
    if (kt0 > 0)
      split = (int)blockIdx.x - __builtin_amdgcn_readfirstlane(
                                    a.bal_on ? bal_owner(bw, G, U, rbg * T)
                                             : attend_owner(rbg * T, U, G));
    const int row0 = rb * C::ROWS;
    const int key_begin = kt0 * BN;
    const int key_end = min(a.n_valid, (kt0 + n_tiles) * BN);
    const char* c_base = reinterpret_cast<const char*>(a.c_kv + (size_t)b * a.geo.ring_tokens * DC);
    const uint16_t* r_base = a.k_r + (size_t)b * a.geo.ring_tokens * DR + kch * 8;
    __syncthreads();  // the previous segment's LDS areas are no longer read

    // queries of this wave's 32 rows, B-operand layout: lane holds row 16 rs + l16, columns
    // 32 ks + 8 qd .. +8
    bf16x8 q[2][KS];
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) {
      const int r = row0 + 32 * rh + 16 * rs + l16;
      const uint16_t* src = a.qcat + ((size_t)b * rows_b + (r < rows_b ? r : 0)) * C::DQK + 8 * qd;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        q[rs][ks] = as_bf16x8(r < rows_b ? ldg16(src + 32 * ks) : u32x4{0, 0, 0, 0});
    }

    // This wave's loads of the tile of keys k0 ..; rows at or past key_end repeat row key_end - 1:
    // finite values whose scores are masked. lim[i mod 4] is load i's offset at the last row.
    const char* tile_base;
    uint32_t tile_lds, lim[4];
    auto dma_begin = [&](int k0, uint16_t* buf) {
      const int k = min(k0, key_end - 1), last = min(key_end - 1 - k, BN - 1);
      tile_base = c_base + (size_t)k * (DC * 2);
      tile_lds = __builtin_amdgcn_readfirstlane(lds_addr(buf) + wave * DC * 2);
#pragma unroll
      for (int i = 0; i < 4; ++i) lim[i] = last * DC * 2 + (coff[i] & (DC * 2 - 1));
    };
    auto dma_c = [&](auto ic) {
      constexpr int i = decltype(ic)::value;
      lds_dma16_min<i * C::NW * DC * 2>(tile_base, coff[i], lim[i & 3], tile_lds);
    };
    auto dma_r = [&](int k0, uint16_t* buf) {
      if (wave < C::RL)
        lds_dma16(r_base + (size_t)min(k0 + krow, key_end - 1) * DR,
                  __builtin_amdgcn_readfirstlane(lds_addr(buf) + BN * DC * 2 + wave * 1024));
    };
    auto dma_tile = [&](int k0, uint16_t* buf) {
      dma_begin(k0, buf);
      for_const<C::CL>(dma_c);
      dma_r(k0, buf);
    };
    auto kread = [&](const uint16_t* buf, int ks) {
      return as_bf16x8(*reinterpret_cast<const u32x4*>(
          &buf[ks < KS - 1 ? kofs[ks & 3] + (ks >> 2) * 128 : kofs_r]));
    };

    f32x16 o[2][DB];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int d = 0; d < DB; ++d) o[x][d] = f32x16{};
    float m_row = kNegInfW;               // running max of row `lane`, the same in every wave
    float ms[2], l_run[2] = {0.f, 0.f};   // score rows 16 rs + l16: running max, this lane's sum

    // keys at or past key_end get -inf; then the row max of this wave's 16 keys, to LDS
    auto mask_tail = [&](int kbase, f32x4 (&s)[2]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool dead = kbase + 16 * kh + 4 * qd + i >= key_end;
#pragma unroll
        for (int rs = 0; rs < 2; ++rs) s[rs][i] = dead ? kNegInfW : s[rs][i];
      }
    };
    auto put_max = [&](const f32x4 (&s)[2]) {
      float v[2];
#pragma unroll
      for (int rs = 0; rs < 2; ++rs)
        v[rs] = quad_max(fmaxf(fmaxf(fmaxf(s[rs][0], s[rs][1]), s[rs][2]), s[rs][3]));
      if (qd < 2) mx[kh][32 * rh + lane] = qd == 0 ? v[0] : v[1];
    };
    // score-row layout of a value held per row
    auto score_rows = [&](float v, int rs) { return __shfl(v, 32 * rh + 16 * rs + l16); };

    dma_tile(key_begin, tile[0]);
    dma_tile(key_begin + BN, tile[1]);
    dma_tile(key_begin + 2 * BN, tile[2]);
    wait_vmcnt<0>();
    __syncthreads();
    if (stamp_step == 0) VMLA_STAMP(a, kStampAttend, 1);
    if (stamp_seg == 1) VMLA_STAMP(a, kStampAttend, 14);

    // scores of tile 0, its row max as the running max
    f32x4 s_cur[2] = {f32x4{}, f32x4{}};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const bf16x8 k = kread(tile[0], ks);
#pragma unroll
      for (int rs = 0; rs < 2; ++rs) s_cur[rs] = mfma16w(k, q[rs][ks], s_cur[rs]);
    }
    if (key_begin + BN > key_end) mask_tail(key_begin, s_cur);
    put_max(s_cur);
    // Operands read ahead: 6 score and 3 value operands (4 and 3: 3610 us, 8 and 3: 3740, 6 and 2:
    // 3530, against 3500 at the shape above).
    constexpr int PF = 6, VA = 3;
    bf16x8 kq[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) kq[i] = kread(tile[1], i);
    __syncthreads();
    m_row = fmaxf(mx[0][lane], mx[1][lane]);
#pragma unroll
    for (int rs = 0; rs < 2; ++rs) ms[rs] = score_rows(m_row, rs);

    uint16_t *p0 = tile[0], *p1 = tile[1], *p2 = tile[2], *p3 = tile[3];
    for (int t = 0; t < n_tiles; ++t) {
      const int kbase = key_begin + t * BN;
      // Tile t+3 goes into tile t-1's buffer, whose last reads precede the last barrier: one load
      // now, the others one by one under the PV product, whose MFMAs take twice as long as the
      // score slots'. A wave that issues its loads in one go waits for those of all four (the
      // compute unit takes in 64 B per cycle) with no other wave on its SIMD to fill the matrix
      // pipe: 3990 us; half of them in the score slots: 3640 us.
      const int k_dma = kbase + 3 * BN;
      dma_begin(k_dma, p3);
      float mx0 = mx[0][lane], mx1 = mx[1][lane];
      f32x4 s_nxt[2] = {f32x4{}, f32x4{}};
      bf16x8 vq[VA + 1], pq[2][2];
      const lds_u16* cur = as_lds(p0);
      auto vread = [&](int j) {  // V operand j: key block j / DB, value block j % DB
        const int kk = j / DB, d = j % DB;
        return join_bf16x8(lds_read_tr(cur + vlo[d] + kk * 16 * DC),
                           lds_read_tr(cur + vhi[d] + kk * 16 * DC));
      };
      // the softmax's slots: the max check (its LDS reads have passed under the slots before),
      // four quarters of the exponentials, the P^T writes; then the barrier
      constexpr int SMAX = 4, SWR = SMAX + 4, SBAR = SWR + 4;
      static_assert(SBAR + 2 < KS, "P^T is read under the last score steps");
      uint32_t pk[2][2];
      auto score_slot = [&](auto ksc) {
        constexpr int ks = decltype(ksc)::value;
        if constexpr (ks == SBAR) {
          // P(t) written; this wave's part of tile t+2 landed (all but this step's one load)
          // (of the operations issued after the P^T writes, only operand reads may pend)
          wait_lgkmcnt<(KS - PF < SBAR ? (KS - PF > SWR + 1 ? KS - PF - SWR - 1 : 0) : SBAR - SWR - 1)>();
          wait_vmcnt<1>();
          bare_barrier();
#pragma unroll
          for (int x = 0; x < 2; ++x)
            pq[0][x] = as_bf16x8(*reinterpret_cast<const u32x4*>(&pbuf[x][0][g][l32][0]));
          vq[0] = vread(0);
        }
        if constexpr (ks > SBAR && ks - SBAR < VA) vq[ks - SBAR] = vread(ks - SBAR);
        if constexpr (ks == SBAR + 1) {
#pragma unroll
          for (int x = 0; x < 2; ++x)
            pq[1][x] = as_bf16x8(*reinterpret_cast<const u32x4*>(&pbuf[x][1][g][l32][0]));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int rs = 0; rs < 2; ++rs) s_nxt[rs] = mfma16w(kq[ks % PF], q[rs][ks], s_nxt[rs]);
        if (ks + PF < KS) kq[ks % PF] = kread(p1, ks + PF);
        if constexpr (ks == 0) dma_c(std::integral_constant<int, 0>{});
        if (ks == SMAX) {
          asm volatile("" : "+v"(mx0), "+v"(mx1));  // not before this slot: the reads' wait
          const float v = fmaxf(mx0, mx1);
          // the same data in every wave, hence the same decision
          if (__builtin_amdgcn_ballot_w64(v > m_row + kLazyMaxW) != 0) {
            const float m_new = fmaxf(m_row, v);
            const float alpha = fast_exp2(m_row - m_new);
            m_row = m_new;
#pragma unroll
            for (int rs = 0; rs < 2; ++rs) {
              ms[rs] = score_rows(m_new, rs);
              l_run[rs] *= score_rows(alpha, rs);
            }
            // through LDS: the accumulators live in accumulation registers
#pragma unroll
            for (int x = 0; x < 2; ++x) {
              const float al = __shfl(alpha, 32 * x + l32);
#pragma unroll
              for (int d = 0; d < DB; ++d) {
                f32x16* slot = reinterpret_cast<f32x16*>(&resc[wave][lane * 16]);
                *slot = o[x][d];
                asm volatile("" ::: "memory");
                f32x16 tmp = *slot;
                tmp *= al;
                *slot = tmp;
                asm volatile("" ::: "memory");
                o[x][d] = *slot;
              }
            }
          }
        }
        if (ks >= SMAX && ks < SMAX + 4) {
          const int rs = (ks - SMAX) >> 1, i = (ks - SMAX) & 1;
          const f32x2 e = {fast_exp2(s_cur[rs][2 * i] - ms[rs]), fast_exp2(s_cur[rs][2 * i + 1] - ms[rs])};
          const bf16x2 h = __builtin_convertvector(e, bf16x2);
          // the sum over the rounded probabilities, as the PV product sees them
          l_run[rs] = __builtin_amdgcn_fdot2_f32_bf16(h, kOnesBf16x2, l_run[rs], false);
          pk[rs][i] = __builtin_bit_cast(uint32_t, h);
        }
        if (ks == SWR) {
          // keys 4 qd .. +4 of key block kh: lane group g = qd mod 2 reads them as its lower
          // (qd < 2: keys 4 g ..) or upper (keys 8 + 4 g ..) half, the order of the V rows
#pragma unroll
          for (int rs = 0; rs < 2; ++rs)
            *reinterpret_cast<u32x2*>(&pbuf[rh][kh][qd & 1][16 * rs + l16][4 * (qd >> 1)]) =
                u32x2{pk[rs][0], pk[rs][1]};
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      for_const<KS>(score_slot);
      auto value_slot = [&](auto jc) {
        constexpr int j = decltype(jc)::value, kk = j / DB, d = j % DB;
        if constexpr (j + VA < 2 * DB) vq[(j + VA) % (VA + 1)] = vread(j + VA);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < 2; ++x) o[x][d] = mfma32(vq[j % (VA + 1)], pq[kk][x], o[x][d]);
        if constexpr (j + 1 < C::CL) dma_c(std::integral_constant<int, j + 1>{});
        if constexpr (j + 1 == C::CL) dma_r(k_dma, p3);
        if constexpr (j == 1) {
          if (kbase + 2 * BN > key_end) mask_tail(kbase + BN, s_nxt);  // near the segment's end
          put_max(s_nxt);
        }
        // the next step's first operands: tile t+2, complete since the barrier above
        if constexpr (j >= 2 * DB - PF) kq[j - (2 * DB - PF)] = kread(p2, j - (2 * DB - PF));
        __builtin_amdgcn_sched_barrier(0);
      };
      for_const<2 * DB>(value_slot);
      s_cur[0] = s_nxt[0];
      s_cur[1] = s_nxt[1];
      const bool stamped = stamp_step >= 200 && stamp_step < 204;
      const uint64_t stream_end = stamped ? VMLA_STAMP_NOW() : 0;
      wait_lgkmcnt<PF>();  // the max, and every read of tile t; the operands of tile t+2 may pend
      bare_barrier();
      if (stamped) {
        VMLA_STAMP(a, kStampAttend, 3 + 2 * (stamp_step - 200));
        VMLA_STAMP_AT(a, kStampAttend, 2 + 2 * (stamp_step - 200), stream_end);
      }
      ++stamp_step;
      uint16_t* tmp = p0;
      p0 = p1;
      p1 = p2;
      p2 = p3;
      p3 = tmp;
    }

    VMLA_STAMP(a, kStampAttend, 10);  // the segment processed last keeps its stamp
    if (stamp_seg == 0) VMLA_STAMP(a, kStampAttend, 12);

    // ---- unnormalized O_lat and (max, sum) of this split ----------------------------------
    wait_vmcnt<0>();  // the last tiles' loads are done before their buffers are reused
    const size_t total_rows = (size_t)a.batch * rows_b;
    const size_t row_base = (size_t)split * total_rows + (size_t)b * rows_b + row0;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      if (row0 + 32 * x + l32 >= rows_b) continue;
      float* op = a.o_part + (row_base + 32 * x + l32) * DC + wave * DB * 32 + 4 * g;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<f32x4*>(op + d * 32 + 8 * i) =
              f32x4{o[x][d][4 * i], o[x][d][4 * i + 1], o[x][d][4 * i + 2], o[x][d][4 * i + 3]};
    }
    const float ls0 = quad_sum(l_run[0]), ls1 = quad_sum(l_run[1]);
    if (qd < 2) mx[kh][32 * rh + lane] = qd == 0 ? ls0 : ls1;
    __syncthreads();
    if (wave == 0 && row0 + lane < rows_b) {
      float* ml = a.ml_part + (row_base + lane) * 2;
      ml[0] = m_row;
      ml[1] = mx[0][lane] + mx[1][lane];
    }
    if (stamp_seg == 0) VMLA_STAMP(a, kStampAttend, 13);
    ++stamp_seg;
  }
  VMLA_STAMP_DRAINED(a, kStampAttend, 11);
  if (a.bal_rec && tid == 0)
    a.bal_state[kBalHead + blockIdx.x] = (uint32_t)(__builtin_amdgcn_s_memrealtime() - bal_t0);
}

}  // namespace

hipError_t launch_latent_attend_wide(const AttendArgs& a, hipStream_t s) {
  // validated by the caller: d_c = 512, d_rope = 32, rows and keys per block as in WideCfg
  hipLaunchKernelGGL(latent_attend_wide_kernel, dim3(a.n_wg), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace vmla
