// Q4_0-weight GEMM in tiles of 32, 64 or 128 rows x 128 columns, or 128 x 256
// (gfx950).  The narrow tiles take the products whose 256 x 256 tiles
// (gemm_q4.hip) would leave the chip idle -- short prompts, few dropped
// chunks, narrow projections; the 128 x 256 ones the large products that do
// not make whole rounds of those.  The results are the same bits as that
// kernel's: each output element is the same sequence of 32-deep MFMAs over
// the same halves.
//
// What bounds it: with few rows the weight stream and the latency of a K
// step, with 128 rows and the chip full the MFMAs, their LDS reads and the
// dequantization, which all want the same issue slots.  So:
//  - Four waves of 32 (or 64) columns share the activation rows in LDS, and
//    two such workgroups fit a CU, so one computes while the other waits at its
//    barrier.  A wave dequantizes only its own columns, into registers: the
//    weights never go back to LDS (the 256-row kernel writes them there), and
//    a lane's MFMA operand is exactly one code dword.
//  - Everything arrives by LDS-DMA (activations, codes and scales), NS - 1
//    stages ahead and waited for by count, so nothing of a stage sits in
//    registers.
//  - The weights are the first MFMA operand, so a lane ends up with four
//    consecutive columns of one row: 16-byte fp32 and 8-byte f16 stores.
//  - The loop is cut into slots of one MFMA; the LDS reads and the
//    dequantization of the next unit and the DMA of a later stage sit in the
//    slots between them (128 rows, one workgroup per CU: a K step 695 -> 638
//    ns against reads and dequantization ahead of the MFMAs).
//
// Measured on one MI355X (us; before: 64-row x 256-column tiles, split over K
// where the grid was small): 17 rows x 4096 x 14336 22.1 -> 15.2, 128 x 28672
// x 4096 82.2 -> 45.3, 256 x 28672 x 4096 130.5 -> 68.4, 512 x 4096 x 14336
// 123 -> 73.5 (818 TFLOP/s), 4979 x 1536 x 8960 213 -> 137 (1000 TFLOP/s).
// 128 x 256 tiles halve the LDS reads and the activation traffic per product:
// with the chip full 1.06-1.2 PFLOP/s against 0.95-1.06 for 128 x 128 and
// 0.97-1.18 for 256 x 256 (4979 x 17920 x 1536: 255 against 288 and 284 us;
// 2048 x 28672 x 4096: 404, 458 and 436).
#include "gemm_rows.h"

#include "q4_dequant.h"
#include "rope.h"

namespace mzk {
namespace {

constexpr int NT = 256;                                  // threads: 4 waves
constexpr int BK = kGemmTileK;
constexpr int NIB_BYTES = kGemmTileN * kGemmTileK / 2;   // code bytes of a packed tile

// MI: 16-row MFMA tiles per wave; NC: 16-column groups per wave (2: 128-column
// tiles, 4: 256).  A stage holds KT 64-wide K tiles of activations, codes and
// scales and is consumed as two units of UK 32-wide blocks; NS stages, as many
// as leave room for two workgroups in a CU's 160 KB (NS * STAGE: 68 KB for 32
// rows, 75 for 64, 63 for 128 x 128 and 75 for 128 x 256).
template <int MI, int NC>
struct RowsTile {
  static constexpr int BM = 16 * MI, BN = 64 * NC;
  static constexpr int KT = MI == 8 ? 1 : 2, UK = KT;
  static constexpr int A_KT = BM * BK * 2, W_KT = BN * BK / 2;
  static constexpr int A_BYTES = KT * A_KT, W_BYTES = KT * W_KT, S_BYTES = 4 * 256;
  static constexpr int STAGE = A_BYTES + W_BYTES + S_BYTES;
  static constexpr int NS = MI == 2 ? 4 : 3;
  static constexpr int AI = BM / 32, WI = NC / 2;             // activation and code loads per wave and K tile
  static constexpr int PER = KT * (AI + WI) + 1;              // loads per wave and stage
  static constexpr int SLOTS = NC * UK * MI;                  // MFMAs of a unit
  static constexpr size_t LDS = (size_t)NS * STAGE;
  static_assert(KT * NC * 16 <= 64, "one lane per scale pair of a stage");
};

// Operands of one unit: dequantized weights of the wave's column groups
// (index NC ks + t) and activation fragments of the row tiles (with four
// groups a fragment is read again, for the next unit, right after its last
// MFMA: no second copy)
template <int MI, int NC>
struct RowsFrag {
  uint32_t w[NC * RowsTile<MI, NC>::UK][4];
  f16x8 a[NC == 4 ? 1 : RowsTile<MI, NC>::UK][NC == 4 ? 1 : MI];
};

// LDS offset (bytes) of logical 16-byte column c of row r (128-byte rows)
__device__ __forceinline__ int swz(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// The rotary epilogue of a wave: acc[i][t] holds columns col(t) + 4 g .. + 3 of
// the tile from column n0 on, for row row0 + 16 i (see the kernel's epilogue).
// Positions and slot offsets come first, the angles a row tile ahead of the
// stores: behind them each read waited for the stores before it (1.5B Q of 8320
// rows 57.1 us, 48.7 now; 1B K/V 64.4 and 56.5, 2048 rows 20.5 and 18.0).
template <int EPI, int MI, int NC, typename Col>
__device__ __forceinline__ void rope_rows(const f32x4 (&acc)[MI][NC], const GemmRope& ea, void* Y, int M, int row0,
                                          int n0, int g, const Col& col) {
  const int half = ea.hd >> 1;
  const int rot = EPI == kEpiRopeQ ? ea.n_valid : ea.n_valid >> 1;   // rotated columns
  int p[MI];
  int64_t off[MI];                                       // < 0: a row that writes nothing
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    p[i] = ea.pos[min(row0 + 16 * i, M - 1)];
    off[i] = EPI == kEpiRopeKV ? ea.kv_off[min(row0 + 16 * i, M - 1)] : 0;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (row0 + 16 * i >= M) off[i] = -1;
    if (off[i] < 0) p[i] = 0;
  }
  float2 cv[2][NC / 2][4];
  auto fetch = [&](int i, float2(&v)[NC / 2][4]) {
#pragma unroll
    for (int t = 0; t < NC; t += 2) {
      const int ct = n0 + col(t);
      if (ct >= rot) continue;
      const float2* cs = ea.rope_cs + (size_t)p[i] * half + ((ct + 4 * g) & (2 * half - 1));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[t / 2][e] = cs[e];
    }
  };
  fetch(0, cv[0]);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (i + 1 < MI) fetch(i + 1, cv[(i + 1) & 1]);
    if (off[i] < 0) continue;
#pragma unroll
    for (int t = 0; t < NC; t += 2) {
      const int ct = n0 + col(t), c0 = ct + 4 * g;
      if (ct < rot) {
        _Float16* y = EPI == kEpiRopeQ ? reinterpret_cast<_Float16*>(Y) + (size_t)(row0 + 16 * i) * ea.n_valid
                                       : reinterpret_cast<_Float16*>(ea.slab + off[i]);
        f16x4 o1, o2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float2 v = cv[i & 1][t / 2][e];
          const float2 q = rope_rotate(acc[i][t][e], acc[i][t + 1][e], v.x, v.y);
          o1[e] = (_Float16)q.x;
          o2[e] = (_Float16)q.y;
        }
        *reinterpret_cast<f16x4_out*>(y + c0) = o1;
        *reinterpret_cast<f16x4_out*>(y + c0 + half) = o2;
      } else if (EPI == kEpiRopeKV) {
        // values: V^T[c][pos % C]; the 16 lanes of a row group are 16
        // activation rows, neighbouring positions in most launches
        const int pc = p[i] & (ea.C - 1);
        uint8_t* vt = ea.slab + off[i] - (int64_t)pc * ea.n_valid + (int64_t)ea.C * ea.n_valid + pc * 2;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int c = c0 + h * half + e;
            if (c < ea.n_valid)
              *reinterpret_cast<_Float16*>(vt + (int64_t)(c - rot) * ea.C * 2) = (_Float16)acc[i][t + h][e];
          }
      }
    }
  }
}

template <int EPI, int MI, int NC>
__global__ __launch_bounds__(NT, 2) void gemm_rows_kernel(
    const _Float16* __restrict__ X, const int32_t* __restrict__ a_rows, int M, int K, const uint8_t* __restrict__ Wp,
    int N, void* __restrict__ Y, int k_steps, GemmRope ea) {
  using T = RowsTile<MI, NC>;
  constexpr int AI = T::AI, WI = T::WI, BN = T::BN;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int n_tiles = N / BN;
  const int b = blockIdx.x, per = (int)gridDim.x / 8;
  const int tile = b < per * 8 ? (b % 8) * per + b / 8 : b;
  const int mt = tile / n_tiles, nt = tile % n_tiles;
  const int split = EPI == kEpiPartial ? (int)blockIdx.y : 0;
  const int ks0 = EPI == kEpiPartial ? split * k_steps : 0;
  const int nk = EPI == kEpiPartial ? min(k_steps, K / BK - ks0) : K / BK;
  constexpr bool ROPE = EPI == kEpiRopeQ || EPI == kEpiRopeKV;
  if (ROPE && nt * BN >= ea.n_valid) return;           // padding columns only
  // The wave's 16-column groups come in pairs, t = 2p and 2p + 1: for the
  // rotary epilogues the two halves of one head's pairs, so a lane holds both;
  // else 32 columns in a row (for SwiGLU, 16 gate columns and their 16 up
  // columns).  Group t starts at column col(t) of the tile.
  const int half = ROPE ? ea.hd >> 1 : 16;
  auto col = [&](int t) {
    const int u = (wave * (NC / 2) + (t >> 1)) * 16;
    return (u / half) * 2 * half + u % half + (t & 1) * half;
  };

  const _Float16* a_src[AI];
#pragma unroll
  for (int i = 0; i < AI; ++i) {
    const int pr = (wave * AI + i) * 8 + (lane >> 3);
    const int lc = (lane & 7) ^ ((pr >> 1) & 7);
    const int row = min(mt * T::BM + pr, M - 1);
    a_src[i] = X + (size_t)(a_rows ? a_rows[row] : row) * K + (size_t)ks0 * BK + lc * 8;
  }
  const uint8_t* wt = Wp + ((size_t)(nt * BN / kGemmTileN) * (K / BK) + ks0) * kGemmTileBytes;
  const int n_in = nt * BN % kGemmTileN;               // first column inside the packed tile
  const uint8_t* w_src = wt + n_in * 32 + wave * WI * 1024 + lane * 16;
  const int sl = lane & (16 * NC - 1);                 // scale pair of column sl % 16 of group sl / 16
  int scol = col(0);
#pragma unroll
  for (int t = 1; t < NC; ++t) scol = (sl >> 4) == t ? col(t) : scol;
  const uint8_t* s_src = wt + NIB_BYTES + (n_in + scol + r) * 4;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void*)lds;
  // load j of stage s: per K tile AI activation loads and the codes, then the
  // scales of the stage (one wait state between each M0 write and the LDS-DMA
  // load that reads it)
  auto dma = [&](int j, int s, uint32_t base) {
    const int kt0 = s * T::KT, kt1 = min(kt0 + T::KT, nk) - 1;   // an odd last K tile stands in for its missing pair
    if (j < T::PER - 1) {
      const int kj = j / (AI + WI), i = j % (AI + WI);
      const int kt = kj ? kt1 : kt0;
      if (i < AI)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(base + kj * T::A_KT +
                                                                                          (wave * AI + i) * 1024),
                     "v"(a_src[i < AI ? i : 0] + kt * BK)
                     : "memory", "m0");
      else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(base + T::A_BYTES + kj * T::W_KT +
                                                                                          (wave * WI + i - AI) * 1024),
                     "v"(w_src + (i < AI ? 0 : i - AI) * 1024 + (size_t)kt * kGemmTileBytes)
                     : "memory", "m0");
    } else {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(base + T::A_BYTES + T::W_BYTES +
                                                                                       wave * 256),
                   "v"(s_src + (size_t)(lane < 16 * NC ? kt0 : kt1) * kGemmTileBytes)
                   : "memory", "m0");
    }
  };
  const int a_off = swz(r, g);                         // of row tile 0, 32-wide block 0
  int w_off[NC];
#pragma unroll
  for (int t = 0; t < NC; ++t) w_off[t] = T::A_BYTES + (col(t) + r) * 32 + g * 4;
  const int s_off = T::A_BYTES + T::W_BYTES + wave * 256 + r * 4;
  uint32_t wq[NC * T::UK], sc[NC];                     // codes and scales of the unit being read
  f16x8 am[NC == 4 ? MI : 1];                          // activation fragments, one copy
  auto read_w = [&](const uint8_t* st, int unit) {
    const int j = T::UK == 2 ? unit : 0, k0 = T::UK == 2 ? 0 : unit;
#pragma unroll
    for (int t = 0; t < NC; ++t) {
#pragma unroll
      for (int ks = 0; ks < T::UK; ++ks)
        wq[NC * ks + t] = *reinterpret_cast<const uint32_t*>(st + w_off[t] + j * T::W_KT + (k0 + ks) * 16);
      sc[t] = *reinterpret_cast<const uint32_t*>(st + s_off + j * NC * 64 + t * 64);
    }
  };
  auto read_a = [&](RowsFrag<MI, NC>& f, const uint8_t* st, int unit, int e) {
    const int j = T::UK == 2 ? unit : 0, ks = (T::UK == 2 ? 0 : unit) + e / MI, i = e % MI;
    const f16x8 v = *reinterpret_cast<const f16x8*>(st + j * T::A_KT + (a_off ^ (ks * 64)) + i * 2048);
    if constexpr (NC == 4)
      am[i] = v;
    else
      f.a[e / MI][i] = v;
  };
  // code pair m of fragment q (see dequant_pair)
  auto deq = [&](RowsFrag<MI, NC>& f, int unit, int e) {
    const int q = e >> 2, m = e & 3;
    const int sh = T::UK == 2 ? 16 * (q / NC) : 16 * unit;
    const _Float16 d = __builtin_bit_cast(_Float16, (uint16_t)(sc[q % NC] >> sh));
    f.w[q][m] = dequant_pair(wq[q], m, f16x2{d, d});
  };

  f32x4 acc[MI][NC];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int t = 0; t < NC; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // One unit: its MFMAs, one per slot, and in the slots between them the LDS
  // reads and the dequantization of the next unit (unit `un` of the stage at
  // st) and DMA loads j0 .. j1 - 1 of stage sd.
  auto unit = [&](const RowsFrag<MI, NC>& f, RowsFrag<MI, NC>& fn, const uint8_t* st, int un, int j0, int j1, int sd,
                  uint32_t base, bool load) {
    constexpr int NA = T::UK * MI, ND = 4 * NC * T::UK, D0 = T::SLOTS / 4 + 1, DS = T::SLOTS - D0;
    read_w(st, un);
#pragma unroll
    for (int i = 0; i < T::SLOTS; ++i) {
      const int q = i / MI, e = i % MI;
      if constexpr (NC == 2) {
#pragma unroll
        for (int x = 0; x < NA; ++x)
          if (x * (T::SLOTS / 2) / NA == i) read_a(fn, st, un, x);
      }
      __builtin_amdgcn_sched_barrier(0);
      f16x8 af;
      if constexpr (NC == 4)
        af = am[e];
      else
        af = f.a[q / NC][e];
      acc[e][q % NC] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
          __builtin_bit_cast(f16x8, uint4{f.w[q][0], f.w[q][1], f.w[q][2], f.w[q][3]}), af, acc[e][q % NC], 0, 0, 0);
      if constexpr (NC == 4) {
        if (q == NC - 1) read_a(fn, st, un, e);
      }
#pragma unroll
      for (int x = 0; x < ND; ++x)
        if (D0 + x * DS / ND == i) deq(fn, un, x);
      const int n = j1 - j0;
#pragma unroll
      for (int x = 0; x < T::PER; ++x)
        if (x < n && x * T::SLOTS / n == i && load) dma(j0 + x, sd, base);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  const int n_st = (nk + T::KT - 1) / T::KT;
  constexpr int JB = (T::PER + 1) / 2;      // loads issued in a stage's second unit; the others in the next unit
  RowsFrag<MI, NC> f0, f1;
  for (int s = 0; s < T::NS && s < n_st; ++s)
    for (int j = 0; j < T::PER; ++j) dma(j, s, __builtin_amdgcn_readfirstlane(lds0 + s * T::STAGE));
  {
    const int rem = min(T::NS - 1, n_st - 1);
    if (rem == T::NS - 1) wait_vm<(T::NS - 1) * T::PER>();
    else if (T::NS > 3 && rem == 2) wait_vm<2 * T::PER>();
    else if (rem == 1) wait_vm<T::PER>();
    else wait_vm<0>();
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_w(lds, 0);
#pragma unroll
  for (int x = 0; x < T::UK * MI; ++x) read_a(f0, lds, 0, x);
#pragma unroll
  for (int x = 0; x < 4 * NC * T::UK; ++x) deq(f0, 0, x);
  int slot = 0, prev = T::NS - 1;
  for (int s = 0; s < n_st; ++s) {
    const int nxt = slot == T::NS - 1 ? 0 : slot + 1;
    const uint8_t* st = lds + slot * T::STAGE;
    unit(f0, f1, st, 1, JB, T::PER, s - 1 + T::NS, __builtin_amdgcn_readfirstlane(lds0 + prev * T::STAGE),
         s > 0 && s - 1 + T::NS < n_st);
    if (T::KT == 2 && 2 * s + 1 >= nk) break;          // an odd last K tile
    // stage s + 1 has landed and every wave has read stage s to its end
    const int rem = min(T::NS - 2, n_st - 2 - s);      // stages after s + 1 that may stay in flight
    if (rem == T::NS - 2) wait_vm<(T::NS - 2) * T::PER>();
    else if (T::NS > 3 && rem == 1) wait_vm<T::PER>();
    else wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    unit(f1, f0, lds + nxt * T::STAGE, 0, 0, JB, s + T::NS, __builtin_amdgcn_readfirstlane(lds0 + slot * T::STAGE),
         s + T::NS < n_st);
    prev = slot;
    slot = nxt;
  }

  // epilogue: lane (r, g) holds columns c + 4 g .. + 3 of each 16-column
  // group for activation row r of each 16-row tile
  if constexpr (ROPE) {
    rope_rows<EPI>(acc, ea, Y, M, mt * T::BM + r, nt * BN, g, col);
    return;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int row = mt * T::BM + i * 16 + r;
    if (row >= M) continue;
#pragma unroll
    for (int t = 0; t < NC; t += 2) {
      const int ct = nt * BN + col(t), c0 = ct + 4 * g;
      if constexpr (EPI == kEpiSwiGLU) {
        f16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = swiglu_f16(acc[i][t][e], acc[i][t + 1][e]);
        *reinterpret_cast<f16x4_out*>(reinterpret_cast<_Float16*>(Y) + (size_t)row * (N / 2) + ct / 2 + 4 * g) = o;
      } else {
        float* y = reinterpret_cast<float*>(Y) + ((size_t)split * M + row) * N + c0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f32x4_out* d = reinterpret_cast<f32x4_out*>(y + 16 * h);
          *d = EPI == kEpiAdd ? *d + acc[i][t + h] : acc[i][t + h];
        }
      }
    }
  }
}

template <int EPI, int MI, int NC>
void launch_t(const _Float16* X, const int32_t* a_rows, int m, int n, int k, const uint8_t* W, void* y, hipStream_t s,
              int n_split, int k_steps, const GemmRope& ea) {
  using T = RowsTile<MI, NC>;
  static const bool ok = [] {   // more than 64 KB of dynamic LDS, once per instantiation
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_rows_kernel<EPI, MI, NC>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)T::LDS);
    return true;
  }();
  (void)ok;
  const int tiles = (n / T::BN) * ((m + T::BM - 1) / T::BM);
  hipLaunchKernelGGL((gemm_rows_kernel<EPI, MI, NC>), dim3(tiles, n_split), dim3(NT), T::LDS, s, X, a_rows, m, k, W, n,
                     y, k_steps, ea);
}

template <int EPI>
void launch_e(const _Float16* X, const int32_t* a_rows, int m, int n, int k, const uint8_t* W, void* y, hipStream_t s,
              int row_tile, int col_tile, int n_split, int k_steps, const GemmRope& ea) {
  switch (row_tile) {
    case 32: launch_t<EPI, 2, 2>(X, a_rows, m, n, k, W, y, s, n_split, k_steps, ea); break;
    case 64: launch_t<EPI, 4, 2>(X, a_rows, m, n, k, W, y, s, n_split, k_steps, ea); break;
    default:
      if (col_tile == 256)
        launch_t<EPI, 8, 4>(X, a_rows, m, n, k, W, y, s, n_split, k_steps, ea);
      else
        launch_t<EPI, 8, 2>(X, a_rows, m, n, k, W, y, s, n_split, k_steps, ea);
      break;
  }
}

}  // namespace

void launch_gemm_rows(const void* x, const int32_t* a_rows, int m, int n, int k, const void* w, int epilogue, void* y,
                      hipStream_t s, int row_tile, int col_tile, int n_split, int k_steps, const GemmRope& ea) {
  const _Float16* X = reinterpret_cast<const _Float16*>(x);
  const uint8_t* W = reinterpret_cast<const uint8_t*>(w);
  switch (epilogue) {
    case kEpiStore: launch_e<kEpiStore>(X, a_rows, m, n, k, W, y, s, row_tile, col_tile, 1, 0, ea); break;
    case kEpiAdd: launch_e<kEpiAdd>(X, a_rows, m, n, k, W, y, s, row_tile, col_tile, 1, 0, ea); break;
    case kEpiSwiGLU: launch_e<kEpiSwiGLU>(X, a_rows, m, n, k, W, y, s, row_tile, col_tile, 1, 0, ea); break;
    case kEpiRopeQ: launch_e<kEpiRopeQ>(X, a_rows, m, n, k, W, y, s, row_tile, col_tile, 1, 0, ea); break;
    case kEpiRopeKV: launch_e<kEpiRopeKV>(X, a_rows, m, n, k, W, y, s, row_tile, col_tile, 1, 0, ea); break;
    default: launch_e<kEpiPartial>(X, a_rows, m, n, k, W, y, s, row_tile, col_tile, n_split, k_steps, ea); break;
  }
}

}  // namespace mzk
