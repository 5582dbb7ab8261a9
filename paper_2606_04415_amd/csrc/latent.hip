// Latent attention (keys 576 wide, values their first 512 columns) over 128
// query rows, for gfx950: decode (128 heads of one token) and prefill (a tile
// of 128 tokens of one head).
//
// What bounds it. Per 32-key tile a work-group does 9.1 MFLOP, 2200 clocks of
// its four matrix cores. A 16-row wave reads one 1 KB operand from LDS per
// 16x16x32 product, which asks for exactly the LDS's 256 bytes a clock and
// leaves nothing for latency; with 32 rows every operand does twice the work.
// 32 rows need 256 accumulators, 144 registers of Q and the scores: one wave
// per SIMD with all 512 registers. With no second wave on the SIMD to fill
// its gaps, one instruction stream has to: operand reads run several products
// ahead, the exponentials of a tile are issued between the score products of
// the next one, and the row maxima of the next tile between the value
// products of this one. Against eight waves of 16 rows: 4096-token prompt of
// 128 heads 2402 -> 2070 us (1.13 PFLOP/s; a loop of nothing but these
// products reaches 1.84), 256 decodes over 1024 to 16384 keys 759 -> 730 us.
#include <float.h>
#include <math.h>

#include <type_traits>
#include <utility>

#include "device_common.h"
#include "kernels.h"
#include "latent_tile.h"

namespace flexattn {

namespace {

typedef __bf16 short2v __attribute__((ext_vector_type(2)));

constexpr int kQK = kLatentQK, kV = kLatentV;
constexpr int kBN = kLatentBN;
constexpr int kNW = 4;                   // waves, 32 query rows each
constexpr int kDC = kQK / 16;            // 16-dim chunks of the score products
constexpr int kACC = kV / 32;            // 32-column blocks of the values
constexpr int kStages = 4;
// Neighbouring 16-byte chunks are swapped in rows 16 to 31, without which the
// 32 rows of a key operand read conflict (key / transposing value reads 233 /
// 200 bytes a clock; without the swap 123 for the keys).
constexpr int kRow = kLatentRow, kTailOff = kLatentTailOff, kStage = kLatentStage, kLoads = kLatentLoads;
// A row's maximum moves only when a tile raises it by more than this many
// log2 units, as in the other row-parallel kernels. A fresher maximum is not
// only a matter of range: a row's largest probability is exactly 1 while it
// is the maximum, and rounded to bf16 otherwise (with 24 units here the error
// of the log-sum-exp against 64 bits is 1.3 times as large).
constexpr float kRescale = 8.0f;
// Prefill tiles of few rows take 16 a wave instead of 32, so that twice as many
// waves share the output's conversion and stores, if they are short enough for
// that to count: 32 rows of 32 keys 9.6 -> 8.6 us, 64 rows of 64 keys 13.1 ->
// 12.1, at 500 keys alike, at 4000 the further waves' LDS reads cost 0.5%.
constexpr int kSpreadRows = 64, kSpreadKeys = 256;
constexpr int kWin = 2048;               // block-table entries held in LDS
constexpr int kLds = kStages * kStage + kWin * 4;
static_assert(kLds <= 160 * 1024, "LDS of a compute unit");

template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

// Matrix products of 32x32x16: lane l = 32h + n supplies row n of A and
// column n of B, 8 contraction slots of half h each, and receives
// D[8i + 4h + r][n] in register 4i + r. Half as many instructions as 16x16x32
// for the same operands leave the wave's other instructions room to issue.
// They are written as instructions so that the accumulators stay in
// accumulation registers and the scores in vector registers (the compiler
// gives all results of a kernel the same kind, and 256 + 32 do not fit one).
// It does not see the products' result latency: every reader of a result
// that is not another product of the same accumulator comes after
// product_wait() or at least four products later (32 clocks each).
typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ void mfma_first(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_vgpr(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_agpr(f32x16& d, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void product_wait() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
// The scores (accumulators) may be read from here on. The wait alone does not
// keep plain reads of them below it: their values have to pass through here.
__device__ __forceinline__ void scores_ready(f32x16& s) { asm volatile("" : "+v"(s)); }
template <int N>
__device__ __forceinline__ void accumulators_ready(f32x16 (&o)[N]) {
#pragma unroll
  for (int a = 0; a < N; ++a) asm volatile("" : "+a"(o[a]));
}

// One element of an accumulator (read this way because the compiler moves whole
// accumulators to vector registers for plain reads of their elements).
__device__ __forceinline__ float acc_read(float a) {
  float v;
  asm("v_accvgpr_read_b32 %0, %1" : "=v"(v) : "a"(a));
  return v;
}

// Scales register R of every accumulator if one of the two rows it holds (ROW
// in the low half of the wave, ROW + 4 in the high half) is set in `rows`, by
// the factors that lanes ROW and ROW + 4 hold in alpha. The branch is inside
// the block because the compiler, given a branch per register, copies all
// accumulators at each. The waits are those between a vector instruction that
// writes a scalar (or alpha) and the one that reads it.
template <int R>
__device__ __forceinline__ void scale_register(f32x16 (&o)[kACC], uint32_t rows, float alpha) {
  constexpr int ROW = 8 * (R >> 2) + (R & 3);
  static_assert(kACC == 16, "operands below");
  float f, t, v[kACC];
  uint32_t s0, s1;
#pragma unroll
  for (int a = 0; a < kACC; ++a) v[a] = o[a][R];
  asm volatile(
      "s_and_b32 %[s0], %[rows], %[bits]\n\t"
      "s_cbranch_scc0 .Lscaled_%=\n\t"
      "v_readlane_b32 %[s0], %[alpha], %[row]\n\t"
      "v_readlane_b32 %[s1], %[alpha], %[row] + 4\n\t"
      "s_nop 1\n\t"
      "v_mov_b32 %[f], %[s0]\n\t"
      "v_mov_b32 %[t], %[s1]\n\t"
      "v_cndmask_b32_e64 %[f], %[f], %[t], %[high]\n\t"
      ".irp reg, %0, %1, %2, %3, %4, %5, %6, %7, %8, %9, %10, %11, %12, %13, %14, %15\n\t"
      "v_accvgpr_read_b32 %[t], \\reg\n\t"
      "v_mul_f32 %[t], %[t], %[f]\n\t"
      "v_accvgpr_write_b32 \\reg, %[t]\n\t"
      ".endr\n\t"
      ".Lscaled_%=:"
      : "+a"(v[0]), "+a"(v[1]), "+a"(v[2]), "+a"(v[3]), "+a"(v[4]), "+a"(v[5]), "+a"(v[6]), "+a"(v[7]), "+a"(v[8]),
        "+a"(v[9]), "+a"(v[10]), "+a"(v[11]), "+a"(v[12]), "+a"(v[13]), "+a"(v[14]), "+a"(v[15]), [f] "=&v"(f),
        [t] "=&v"(t), [s0] "=&s"(s0), [s1] "=&s"(s1)
      : [rows] "s"(rows), [alpha] "v"(alpha), [high] "s"(0xFFFFFFFF00000000ull), [bits] "n"(0x11u << ROW), [row] "n"(ROW)
      : "scc");
#pragma unroll
  for (int a = 0; a < kACC; ++a) o[a][R] = v[a];
}

// Max over the two halves of the wave, on the VALU.
__device__ __forceinline__ float half_max(float v) { return swap32_combine_max(v); }
__device__ __forceinline__ float half_sum(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto t = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(t[0]) + __uint_as_float(t[1]);
}

}  // namespace

// DECODE: work-group (piece, group of 128 heads); else (tile of 128 tokens,
// query head).
template <bool DECODE, int P>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void latent_kernel(AttnParams p) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
  int* s_pt = reinterpret_cast<int*>(lds + kStages * kStage);
  int item = int(blockIdx.x), col = int(blockIdx.y);
  if (!DECODE && p.xcd_remap) {
    // Head h on XCD h % 8 for all its tiles, tiles longest first: each XCD's
    // L2 then works on one stretch of the keys.
    const int x = int(blockIdx.x) & 7, j = int(blockIdx.x) >> 3, hp8 = p.grid_y / 8;
    item = j / hp8;
    col = (j % hp8) * 8 + x;
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int it = 8 * (DECODE ? scalar_word(p.order, item) : item);
  const int seq = scalar_word(p.items, it);
  const int L = scalar_word(p.seq_lens, seq);
  const int q0 = scalar_word(p.qsl, seq);
  const int nq = scalar_word(p.qsl, seq + 1) - q0;
  const int32_t* bt_row = p.bt + int64_t(seq) * p.bt_stride;

  // Query token, head and key limit of the lane's rows; rows past the tile's
  // end repeat the wave's first row and are not written. wave_limit: end of
  // the keys any row of the wave sees; wave_full: every row sees those below.
  const int it2 = scalar_word(p.items, it + 2), it3 = scalar_word(p.items, it + 3), it4 = scalar_word(p.items, it + 4);
  int key_begin, key_end, head_kv, wave_limit, wave_full;
  bool wave_on = true;
  int wave_rows = 32;   // rows of the tile that a wave takes
  int row_limit;
  const uint16_t* q_row;
  if constexpr (DECODE) {
    key_begin = it3;
    key_end = min(it4, L);
    head_kv = (col * p.rows_per_wg) / p.G;
    q_row = p.q + (int64_t(q0) * p.Hq + col * p.rows_per_wg + w * 32 + n) * kQK;
    row_limit = wave_limit = wave_full = key_end;
  } else {
    key_begin = 0;
    key_end = it4;
    head_kv = col / p.G;
    if (it3 - it2 <= kSpreadRows && it4 <= kSpreadKeys) wave_rows = 16;
    const int wr0 = it2 + w * wave_rows;
    const int wr1 = min(it3, wr0 + wave_rows);
    wave_on = wr0 < it3;
    const int lr = wr0 + n < wr1 ? wr0 + n : wr0;
    q_row = p.q + (int64_t(q0 + (wave_on ? lr : it2)) * p.Hq + col) * kQK;
    row_limit = L - nq + lr + 1;
    wave_limit = wave_on ? L - nq + wr1 : 0;
    wave_full = L - nq + wr0 + 1;
  }

  // Q as the B operand of S^T = K Q^T.
  u32x4 qop[kDC];
#pragma unroll
  for (int c = 0; c < kDC; ++c) qop[c] = load16(q_row + 8 * h + 16 * c);

  f32x16 o[kACC];
  float m = -FLT_MAX;   // lowest finite value: masked keys then add zeros with no guard
  float l = 0.f, alpha = 1.f;
#pragma unroll
  for (int a = 0; a < kACC; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float z;
      asm volatile("v_accvgpr_write_b32 %0, 0" : "=a"(z));
      o[a][r] = z;
    }

  // Tiles past the window get empty resources: their loads are issued all the
  // same between the score products, where a branch per load would cost more.
  const LatentLoader<P, true> loader(p, head_kv, lds, w, lane);

  // Operand reads: stage base + per-lane offset + immediate. Value block cv
  // covers 32 columns, vcol(cv) + 0..15 in lanes n < 16 and + 64..79 in the
  // others (the 128 bytes between them keep the reads conflict free).
  const uint32_t k_off = uint32_t(n * kRow + 16 * (h ^ (n >> 4)));
  uint32_t k_tail[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) k_tail[c] = uint32_t(kTailOff + n * 128 + 16 * ((2 * c + h) ^ ((n >> 1) & 7)));
  uint32_t v_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
    v_off[ks] = uint32_t((16 * ks + 4 * h + ((lane & 15) >> 2)) * kRow + 128 * (n >> 4) + ((8 * (n & 3)) ^ (16 * ks)));
  auto kread = [&](const uint8_t* stage, int c) {
    return c < 32 ? *reinterpret_cast<const u32x4*>(stage + k_off + 32 * c)
                  : *reinterpret_cast<const u32x4*>(stage + k_tail[c & 3]);
  };
  auto vcol = [](int cv) { return 128 * (cv >> 2) + 16 * (cv & 3); };
  // Keys 16ks + 4h + 0..3 and 16ks + 8 + 4h + 0..3 of value block cv.
  auto vread = [&](const uint8_t* stage, int cv, int ks) {
    const u32x2 lo = lds_read_tr16(reinterpret_cast<const uint16_t*>(stage + v_off[ks] + 2 * vcol(cv)));
    const u32x2 hi = lds_read_tr16(reinterpret_cast<const uint16_t*>(stage + v_off[ks] + (8 * kRow + 2 * vcol(cv))));
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  };
  auto stage_of = [&](int t) { return lds + __builtin_amdgcn_readfirstlane((t & (kStages - 1)) * kStage); };

  // Scores of one tile (register 4i + r: key 8i + 4h + r, row n), with `side`
  // called between the products. Reads run kAhead products ahead.
  constexpr int kAhead = 6;
  auto scores = [&](const uint8_t* stage, f32x16& s, auto&& side) {
    u32x4 kb[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) kb[i] = kread(stage, i);
    __builtin_amdgcn_sched_barrier(0);
    static_for<kDC>([&](auto ic) {
      constexpr int i = ic;
      if constexpr (i == 0) mfma_first(s, kb[i % kAhead], qop[i]);
      else mfma_vgpr(s, kb[i % kAhead], qop[i]);
      if constexpr (i + kAhead < kDC) kb[i % kAhead] = kread(stage, i + kAhead);
      side(ic);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Exponents of a tile: x = s * scale - m, with the row's maximum moved
  // (and alpha, its accumulators' factor, set) only when the tile raises it
  // by more than kRescale.
  float x[16];
  uint32_t moved_rows = 0;   // rows of the wave whose accumulators are due their factor
  auto mask = [&](f32x16& s, int kc0) {
#pragma unroll
    for (int e = 0; e < 16; ++e) s[e] = kc0 + 8 * (e >> 2) + 4 * h + (e & 3) < row_limit ? s[e] : -INFINITY;
  };
  float cmax;
  auto row_max = [&](const f32x16& s, int half) {
    float mx = half ? cmax : s[0];
#pragma unroll
    for (int e = 0; e < 8; ++e) mx = fmaxf(mx, s[8 * half + e]);
    cmax = mx;
  };
  auto new_max = [&]() {
    cmax = half_max(cmax) * p.scale_log2;
    const bool need = cmax > m + kRescale;
    const bool moved = need && m != -FLT_MAX;   // before its first visible key a row's accumulators are zero
    const float m_new = need ? cmax : m;
    alpha = fast_exp2(m - m_new);   // 1 if unchanged
    m = m_new;
    l *= alpha;   // the sums of the tiles before; the accumulators follow in do_rescale
    moved_rows = uint32_t(__builtin_amdgcn_ballot_w64(moved));   // (both halves hold the same rows)
  };
  auto exponent = [&](const f32x16& s, int e) { x[e] = fmaf(s[e], p.scale_log2, -m); };

  // Probabilities 2^x as the bf16 A operand of P V, and their row sums.
  u32x4 pop[2];
  float pe;
  auto prob_lo = [&](int j) { pe = fast_exp2(x[2 * j]); };
  auto prob_hi = [&](int j) {   // j = 0..7: keys of registers 2j, 2j + 1
    const uint32_t pk = pack_bf16x2(pe, fast_exp2(x[2 * j + 1]));
    pop[j >> 2][j & 3] = pk;
    l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(short2v, pk), __builtin_bit_cast(short2v, 0x3F803F80u), l, false);
  };
  // Only registers of a row that moved are scaled, 48 instructions each (an
  // accumulation register passes through a vector register to be
  // multiplied): all 16 cost 3000 clocks, more than a tile, and usually one
  // or two of the 32 rows move.
  auto do_rescale = [&]() {
    product_wait();
    accumulators_ready(o);
    static_for<16>([&](auto rc) { scale_register<rc>(o, moved_rows, alpha); });
    product_wait();
  };

  // O += P V, with `side` called between the products.
  auto values = [&](const uint8_t* stage, auto&& side) {
    u32x4 vb[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) vb[i] = vread(stage, i >> 1, i & 1);
    asm volatile("s_nop 1" : "+v"(pop[0]), "+v"(pop[1]));
    __builtin_amdgcn_sched_barrier(0);
    static_for<2 * kACC>([&](auto ic) {
      constexpr int i = ic;
      mfma_agpr(o[i >> 1], pop[i & 1], vb[i % kAhead]);
      if constexpr (i + kAhead < 2 * kACC) vb[i % kAhead] = vread(stage, (i + kAhead) >> 1, i & 1);
      side(ic);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto nothing = [](auto) {};

  // Windows of kWin block-table entries (one in the usual case); the pipeline
  // drains between windows. Iteration t finds the scores of tile t done,
  // waits for tile t + 1, passes one barrier (every wave is done with tile
  // t - 1, whose stage takes tile t + 3), forms the scores of tile t + 1
  // beside the probabilities of tile t, then adds tile t's values beside the
  // maxima of tile t + 1.
  const int last_page = key_end > 0 ? (key_end - 1) / P : 0;
  for (int wk0 = key_begin; wk0 < key_end; wk0 += kWin * P) {
    const int wk1 = min(key_end, wk0 + kWin * P);
    const int pt_base = wk0 / P;
    lds_barrier();
    for (int i = tid; i <= (wk1 - 1) / P - pt_base; i += kNW * 64) s_pt[i] = bt_row[min(pt_base + i, last_page)];
    wait_vmem_all();   // Q too; from here vmcnt counts tile loads only
    lds_barrier();
    const int ntiles = (wk1 - wk0 + kBN - 1) / kBN;
    const int mine = wave_on ? max(0, min(ntiles, (wave_limit - wk0 + kBN - 1) / kBN)) : 0;
    // Page of the wave's rows of tile t (rows past the window: its last page).
    auto page_at = [&](int t) { return s_pt[min(wk0 + t * kBN + 8 * w, wk1 - 1) / P - pt_base]; };
    auto load_tile = [&](int t) {
      const i32x4 s = loader.source(wk0 + t * kBN, wk1, __builtin_amdgcn_readfirstlane(page_at(t)));
#pragma unroll
      for (int j = 0; j < kLoads; ++j) loader.load_one(s, t & (kStages - 1), j);
    };
    // Tile t + 1 of iteration t (or tile 0 here) has landed once at most the
    // loads of the tiles after it are outstanding. Close to the end those may
    // not have been issued: then for all.
#pragma unroll
    for (int t = 0; t < kStages - 1; ++t)
      if (t < ntiles) load_tile(t);
    if (ntiles > 2) wait_vmem<2 * kLoads>();
    else wait_vmem_all();
    lds_barrier();
    auto wait_next = [&](int t) {
      if (t + 2 < ntiles) wait_vmem<kLoads>();
      else wait_vmem_all();
    };
    f32x16 s;
    if (mine > 0) {
      scores(stage_of(0), s, nothing);
      product_wait();
      scores_ready(s);
      if (wk0 + kBN > wave_full) mask(s, wk0);
      row_max(s, 0);
      row_max(s, 1);
      new_max();
#pragma unroll
      for (int e = 0; e < 16; ++e) exponent(s, e);
    }
    int t = 0;
    for (; t < mine; ++t) {
      wait_next(t);
      lds_barrier();
      if (t + 1 < mine) {
        const int pgv = page_at(t + 3);
        i32x4 src;
        scores(stage_of(t + 1), s, [&](auto ic) {
          constexpr int i = ic;
          if constexpr (i == 1) src = loader.source(wk0 + (t + 3) * kBN, wk1, __builtin_amdgcn_readfirstlane(pgv));
          if constexpr (i % 4 == 2) loader.load_one(src, (t + 3) & (kStages - 1), i / 4);
          if constexpr (i % 4 == 1 && i < 32) prob_lo(i / 4);
          if constexpr (i % 4 == 3 && i < 32) prob_hi(i / 4);
        });
      } else {   // the wave's last tile: s stays, and its maxima move nothing when formed again
        if (t + 3 < ntiles) load_tile(t + 3);
        // (opaque, or the compiler forms both branches' exponentials ahead of the branch)
#pragma unroll
        for (int e = 0; e < 16; ++e) asm volatile("" : "+v"(x[e]));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          prob_lo(j);
          prob_hi(j);
        }
      }
      if (moved_rows) do_rescale();
      const int kc1 = wk0 + (t + 1) * kBN;
      if (kc1 + kBN > wave_full) {
        product_wait();
        scores_ready(s);
        mask(s, kc1);
      }
      values(stage_of(t), [&](auto ic) {
        constexpr int i = ic;
        if constexpr (i == 4) {   // four products after the last one of the scores
          scores_ready(s);
          row_max(s, 0);
        }
        if constexpr (i == 5) row_max(s, 1);
        if constexpr (i == 6) new_max();
        if constexpr (i >= 8 && i < 24) exponent(s, i - 8);
      });
    }
    for (; t < ntiles; ++t) {   // past this wave's rows: loads and barriers only
      wait_next(t);
      lds_barrier();
      if (t + 3 < ntiles) load_tile(t + 3);
    }
    wait_vmem_all();   // nothing may land in LDS after the work-group ends
  }

  // Epilogue: register 4i + r of a lane holds row 8i + 4h + r of the wave.
  product_wait();
  accumulators_ready(o);
  lds_barrier();   // the stages are free: output rows pass through them
  if (!wave_on) return;
  const float ltot = half_sum(l);
  const int row0 = w * wave_rows;   // the wave's first row of the tile; the lane's row of m and l is row0 + n
  if (DECODE && it2 > 1) {   // a split's partial
    const int64_t srow0 = (int64_t(scalar_word(p.items, it + 7)) * int(gridDim.y) + col) * p.rows_per_wg;
    const int vlane = (n & 15) + 64 * (n >> 4);   // column of the lane in a value block
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float* dst = p.ws_o + (srow0 + row0 + 8 * (r >> 2) + 4 * h + (r & 3)) * kV + vlane;
#pragma unroll
      for (int cv = 0; cv < kACC; ++cv) dst[vcol(cv)] = acc_read(o[cv][r]);
    }
    if (h == 0) {
      p.ws_stats[(srow0 + row0 + n) * 2] = m;
      p.ws_stats[(srow0 + row0 + n) * 2 + 1] = ltot;
    }
    return;
  }
  const int64_t out0 = DECODE ? int64_t(q0) * p.Hq + int64_t(col) * p.rows_per_wg : int64_t(q0 + it2) * p.Hq + col;
  const int row_step = DECODE ? 1 : p.Hq;   // output rows between neighbouring rows of the tile
  const int rows = DECODE ? 32 : min(wave_rows, it3 - it2 - row0);   // of the wave
  if (h == 0 && n < rows && p.lse) p.lse[out0 + int64_t(row0 + n) * row_step] = (m + log2f(ltot)) * kLn2;
  // Rows leave through LDS, eight at a time: a lane writes the columns it holds
  // of one row in four neighbouring value blocks (8 bytes), and a transposing
  // read gives it four neighbouring columns of that row, so that a store
  // instruction covers two rows of 256 contiguous bytes. Two bytes a lane
  // straight from the registers, four times as many stores, bound short calls:
  // a decode over 20 keys 13.0 -> 11.5 us, a 128-token prompt 19.2 -> 18.3.
  // (Four rows of 128 bytes in one instruction, neighbouring lanes in
  // different rows, are slower than either: 15.7 and 22.5.)
  constexpr int kOutBuf = 16 * 512;   // 16 reads of 64 lanes x 8 bytes, twice
  static_assert(kNW * 2 * kOutBuf <= kStages * kStage, "output rows fit the stages");
  uint8_t* buf = lds + w * 2 * kOutBuf;
  const uint32_t rd = uint32_t(128 * (lane >> 4) + 8 * (4 * (lane & 3) + ((lane & 15) >> 2)));
  const int col0 = 64 * (n >> 4) + 16 * (lane & 3) + 4 * ((lane & 15) >> 2);
  const float inv_n = 1.f / ltot;
  static_for<4>([&](auto ic) {
    constexpr int i = ic;
    if (8 * i >= rows) return;
    uint8_t* half_buf = buf + (i & 1) * kOutBuf;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float inv = shfl_f(inv_n, 8 * i + 4 * h + r);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int e = 4 * i + r;
        const u32x2 d = {pack_bf16x2(acc_read(o[4 * c][e]) * inv, acc_read(o[4 * c + 1][e]) * inv),
                         pack_bf16x2(acc_read(o[4 * c + 2][e]) * inv, acc_read(o[4 * c + 3][e]) * inv)};
        *reinterpret_cast<u32x2*>(half_buf + (4 * r + c) * 512 + 8 * lane) = d;
      }
    }
    wave_lds_sync();
    u32x2 v[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        v[r][c] = lds_read_tr16(reinterpret_cast<const uint16_t*>(half_buf + rd + (4 * r + c) * 512));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 8 * i + 4 * h + r;
      uint16_t* dst = p.out + (out0 + int64_t(row0 + row) * row_step) * kV + col0;
      if (row < rows) {
#pragma unroll
        for (int c = 0; c < 4; ++c) *reinterpret_cast<u32x2*>(dst + 128 * c) = v[r][c];
      }
    }
  });
}

template <bool DECODE, int P>
static hipError_t launch_latent_t(const AttnParams& p, dim3 grid, hipStream_t stream) {
  auto kern = latent_kernel<DECODE, P>;
  const hipError_t e = set_dynamic_lds(reinterpret_cast<const void*>(kern), kLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid, dim3(kNW * 64), kLds, stream, p);
  return hipGetLastError();
}

hipError_t launch_latent128(const AttnParams& p, bool decode, dim3 grid, hipStream_t stream) {
  if (p.P == 16) return decode ? launch_latent_t<true, 16>(p, grid, stream) : launch_latent_t<false, 16>(p, grid, stream);
  if (p.P == 64) return decode ? launch_latent_t<true, 64>(p, grid, stream) : launch_latent_t<false, 64>(p, grid, stream);
  return hipErrorInvalidValue;
}

}  // namespace flexattn
