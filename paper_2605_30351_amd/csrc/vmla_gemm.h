// The tile loop of the bf16 GEMMs: out^T[o][token] = A[o][:] . B[token][:], a TT-token x TO-output
// tile per workgroup with MFMA 32x32x16 (A = weight rows, B = token rows).
//
// WT x WO waves, each NB x 32 tokens by MO x 32 outputs. An MFMA takes 32 cycles of its SIMD, in
// which the compute unit's LDS delivers 2 KB to each of its four SIMDs, the size of two operand
// blocks; a wave reads (NB + MO) KB per NB MO MFMAs. The contraction streams through ST stages of 32
// columns (token rows, then weight rows, in 16-byte chunks whose index is XOR-ed with a function of
// the row, so that the 32-row operand reads are conflict-free), filled ST - 1 stages ahead by direct
// global-to-LDS loads. Every step's operands are read from LDS one step ahead, those of a stage's
// first step before the barrier between the stages: the barrier of stage i publishes stage i + 1.
#pragma once
#include <type_traits>

#include "vmla_device.h"

namespace vmla {

struct GemmRows {
  const uint16_t* first;
  int more;
};

template <int WT_, int WO_, int NB_, int MO_, int ST_>
struct GemmTile {
  static constexpr int WT = WT_, WO = WO_, NB = NB_, MO = MO_, ST = ST_;
  static constexpr int KC = 32;                     // columns per stage
  static constexpr int NW = WT * WO, NT = NW * 64;
  static constexpr int TT = WT * NB * 32, TO = WO * MO * 32, ROWS = TT + TO;
  static constexpr int CPR = KC / 8;                // chunks per row
  static constexpr int LPW = ROWS * CPR / 64 / NW;  // 1 KB loads per wave and stage
  static constexpr int STAGE = ROWS * KC;           // elements
  static constexpr int KS = KC / 16;                // MFMA steps per stage
  static_assert(ROWS * CPR % (64 * NW) == 0 && LPW % KS == 0, "stage loads split evenly over the waves");
  static_assert(ST >= 3, "lookahead");
  // chunk c of row r sits at c ^ swz(r)
  __device__ static constexpr int swz(int r) { return (r >> 2) & 3; }

  // acc[nb][m]: tokens 32 (NB wt + nb) .. and outputs 32 (MO wo + m) .. of the tile, wave = wt +
  // WT wo. group(r) describes the source of the 16 tile rows from r on (tokens 0 .. TT - 1, then
  // outputs): the first row's pointer and the number of rows that may be read after it (later ones
  // repeat the last), row stride ld elements. The stages are free again after a barrier.
  template <class Group>
  __device__ static __forceinline__ void run(uint16_t* stage, int nchunks, int ld, Group&& group,
                                             f32x16 (&acc)[NB][MO]) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wt = wave % WT, wo = wave / WT;
    const int g = lane >> 5, l32 = lane & 31;
    const uint16_t* src[LPW];  // uniform
    uint32_t voff[LPW];
    for_const<LPW>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      const int r0 = (wave + NW * i) * (64 / CPR), r = r0 + lane / CPR;
      const GemmRows q = group(r0);
      src[i] = q.first;
      voff[i] = (uint32_t)(min(lane / CPR, q.more) * ld + ((lane % CPR) ^ swz(r)) * 8) * 2;
    });
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(stage) + wave * 1024);
    uint32_t koff = 0;  // byte offset of the chunk being loaded
    auto issue = [&](auto ic, int s) {  // load i of that chunk into stage slot s
      constexpr int i = decltype(ic)::value;
      lds_dma16_add<NW * i * 1024>(src[i], voff[i], koff,
                                   __builtin_amdgcn_readfirstlane(lds0 + s * STAGE * 2));
    };
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int m = 0; m < MO; ++m) acc[nb][m] = f32x16{};
#pragma unroll
    for (int c = 0; c < ST - 1; ++c)
      if (c < nchunks) {
        for_const<LPW>([&](auto ic) { issue(ic, c); });
        koff += KC * 2;
      }

    // operand rows wt (wo) .. + l32, chunk 2 ks + g: the XOR of the row is the same for every block
    const int b0 = (wt * NB * 32 + l32) * KC, a0 = (TT + wo * MO * 32 + l32) * KC;
    bf16x8 bx[2][NB], aw[2][MO];
    // operand k of step ks: in the order in which the MFMAs below need them
    auto read = [&](const uint16_t* st, int ks, int k) {
      const int off = ((2 * ks + g) ^ swz(l32)) * 8;
      if (k >= 1 && k <= NB)
        bx[ks & 1][k - 1] = as_bf16x8(*reinterpret_cast<const u32x4*>(&st[b0 + (k - 1) * 32 * KC + off]));
      else {
        const int m = k == 0 ? 0 : k - NB;
        aw[ks & 1][m] = as_bf16x8(*reinterpret_cast<const u32x4*>(&st[a0 + m * 32 * KC + off]));
      }
    };
    if (nchunks >= ST - 1) wait_vmcnt<(ST - 2) * LPW>();
    else wait_vmcnt<0>();
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NB + MO; ++k) read(stage, 0, k);
    int slot = 0;  // stage slot of chunk i
    for (int i = 0; i < nchunks; ++i) {
      const int next = slot + 1 == ST ? 0 : slot + 1, fill = slot == 0 ? ST - 1 : slot - 1;
      if (i + ST - 1 <= nchunks) wait_vmcnt<(ST - 3) * LPW>();
      else wait_vmcnt<0>();
      // chunk i+1 is in LDS for every wave; chunk i-1 is no longer read
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      const bool more = i + ST - 1 < nchunks;
      for_const<KS>([&](auto ksc) {
        constexpr int ks = decltype(ksc)::value, X = NB * MO, R = NB + MO, D = LPW / KS;
        // the next step's operands; past the last chunk a stale stage, never used
        const uint16_t* st = stage + (ks + 1 < KS ? slot : next) * STAGE;
        for_const<X>([&](auto xc) {
          constexpr int x = decltype(xc)::value, m = x / NB, nb = x % NB;
          __builtin_amdgcn_sched_barrier(0);
          acc[nb][m] = mfma32(aw[ks & 1][m], bx[ks & 1][nb], acc[nb][m]);
#pragma unroll
          for (int k = 0; k < R; ++k)
            if (k * X / R == x) read(st, (ks + 1) % KS, k);
          for_const<D>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            if constexpr ((2 * j + 1) * X / (2 * D) == x)
              if (more) issue(std::integral_constant<int, ks * D + j>{}, fill);
          });
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      koff += KC * 2;
      slot = next;
    }
  }
};

}  // namespace vmla
