// Projections of the DiT block: out = epilogue(A . W^T + bias).
//
// bf16: one 256-thread workgroup per compute unit runs a sequence of output
// tiles on the gfx950 matrix cores, fp32 accumulation.  Each of the 4 waves
// (one per SIMD) owns a quarter of the tile, at most 128 x 128, whose
// accumulators live in the accumulation registers.
//
// The matrix instruction is v_mfma_f32_16x16x32_bf16.  These kernels run at
// the board's power limit, and with random operands this shape sustains
// 2.03-2.05 PFLOP/s on the whole chip where v_mfma_f32_32x32x16_bf16 sustains
// 1.78 (register-only loops, 256 x 4 waves; with zeros both reach 2.4).  The
// QKV projection at 75,600 x 15,360 x 5,120 went from 8.9 to 8.4 ms with the
// instruction alone.
//
// The K loop runs in steps of 64: a step's operand tiles are rows of 128 B,
// i.e. whole cache lines.  They go straight from global memory into LDS
// (buffer loads with the lds modifier), into two rings of slots, one per
// operand: no staging registers and no LDS stores, so the loop is 128 MFMAs,
// 32 fragment reads and 16 loads per step for a 256 x 256 tile.  One operand
// (X) has R slots and the other (Y) R + 1: that fills the 160 KiB of LDS with
// 256 x 256 tiles (R = 2) and keeps 1.5 to 2 steps in flight.  A step is two
// halves of 32 in K.  During the MFMAs of a half, the fragments of the next
// half are read; at the barrier between the halves of step s every wave has
// read all of step s and the loads of step s + 1 have landed, so the slot of
// X(s) is refilled with X(s + R) right after it, and the slot of Y(s) with
// Y(s + R + 1) in the first half of step s + 1.  The load cursor runs on into
// the workgroup's next tile, which therefore starts with its first steps in
// LDS; past the last tile it loads nothing (an empty descriptor).
//
// The 16-byte chunks of each 128-byte LDS row are XOR-swizzled so fragment
// reads are free of bank conflicts.  The kernel computes C^T blocks (W as the
// MFMA A operand) so that a lane holds four consecutive output columns of one
// row.  Every tile shape adds up an output element in the same order (one
// chain of 32-wide products, K ascending), so results do not depend on the
// shape: a row of a packed batch has the same bits as alone.
//
// Measured against the former kernel (32x32x16, register-staged loads), the
// builds timed in turn, with the fused epilogues: 75,600 x 15,360 x 5,120
// 8.69 -> 8.28 ms (1.44 PFLOP/s); 4,096 x 12,288 x 3,072 (GELU) 257 -> 224
// us; 4,096 x 3,072 x 12,288 246 -> 210 us; 4,096 x 9,216 x 3,072 189 -> 161
// us; 1,024 x 3,072 x 3,072 63 -> 27 us; 1,024 x 3,072 x 12,288 171 -> 81 us.
// These are repeated launches, whose weights come from the caches.  With weights
// from memory, as in a model whose blocks do not fit the 256 MB last-level
// cache, few rows take longer: 1,024 x 3,072 x 3,072 66 -> 35 us, x 12,288 193
// -> 117 us (4,096 rows: within 3% of the times above).
//
// fp32 (the small exact configuration): see gemm_f32_nt.
#include <atomic>
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace dit {

namespace {

constexpr int BK = 64;                              // K step
constexpr int kWaves = 4;                           // 2 x 2 waves
constexpr int kThreads = 64 * kWaves;
constexpr int kRowBytes = BK * 2;                   // 128 B: one full cache line per tile row
constexpr int kXcds = 8;                            // gfx950: 8 XCDs, workgroups dispatched round-robin

// gelu_tanh(z) = z (1 + tanh u) / 2 = z / (1 + e^(-2u)), u = sqrt(2/pi) (z + 0.044715 z^3)
__device__ __forceinline__ float gelu_tanh(float z) {
  const float k0 = 0.7978845608028654f;  // sqrt(2/pi)
  const float k1 = 0.044715f;
  const float u = k0 * fmaf(k1 * z, z * z, z);
  const float e = __builtin_amdgcn_exp2f(-2.0f * 1.4426950408889634f * u);   // inf for u << 0: z / inf = 0
  return z * __builtin_amdgcn_rcpf(1.0f + e);
}

// Tile sequence of a workgroup.  Each XCD owns a contiguous range of logical
// tiles (the dispatcher places workgroup b on XCD b mod 8); the workgroups of
// one XCD take its tiles round-robin, so at any time they work on adjacent
// tiles.  Logical tiles are rastered in groups of group_m tile rows, so the
// tiles resident on one XCD share A and W panels in its L2 (see raster()).
struct TileSeq {
  int first, stride, count;   // logical tiles first + stride * it, it < count
  int tiles_m, tiles_n, group_m;
  __device__ void coords(int it, int& tm, int& tn) const {
    const int t = first + stride * it;
    const int width = group_m * tiles_n;
    const int group = t / width;
    const int first_m = group * group_m;
    const int gsize = min(tiles_m - first_m, group_m);
    const int r = t - group * width;
    tm = first_m + r % gsize;
    tn = r / gsize;
  }
};

__device__ __forceinline__ TileSeq tile_seq(int b, int nb, int tiles_m, int tiles_n, int group_m) {
  const int tiles = tiles_m * tiles_n;
  const int per_xcd = (tiles + kXcds - 1) / kXcds;
  const int x = b % kXcds, slot = b / kXcds, wgs = nb / kXcds;
  const int lo = x * per_xcd, hi = min(tiles, lo + per_xcd);
  TileSeq q;
  q.first = lo + slot;
  q.stride = wgs;
  q.count = q.first < hi ? (hi - q.first + wgs - 1) / wgs : 0;
  q.tiles_m = tiles_m;
  q.tiles_n = tiles_n;
  q.group_m = group_m;
  return q;
}

// 16-byte chunk swizzle of a 128-byte LDS row: the 16 lanes that read 16
// consecutive rows at one logical chunk touch, with rows 2t and 2t + 1 in
// different halves of a 256-byte bank window and the physical chunk c ^ t
// different for the 8 values of t, 16 distinct bank groups.
__device__ __forceinline__ int row_swizzle(int r) { return (r >> 1) & 7; }

// Raw buffer descriptor over `bytes` bytes from `base`.  The hardware's range
// check covers the lane offset only (not the scalar offset), so a load
// returns zeros where its lane offset is past the end; the loads below carry
// every row offset in the lane offset.
__device__ __forceinline__ u32x4 make_desc(const void* base, int64_t bytes) {
  const uint32_t n = bytes > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)(bytes < 0 ? 0 : bytes);
  const uint64_t p = (uint64_t)base;
  return u32x4{(uint32_t)p, (uint32_t)(p >> 32) & 0xFFFFu, n, 0x00020000u};
}

// 16 bytes per lane from global memory straight into LDS: lane i writes LDS
// bytes lds + 16 i .. +15.  Inline assembly, so the compiler does not make
// later LDS reads wait for it; completion is waited for by hand.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds16(const u32x4& desc, int voff, int soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(lds), "v"(voff), "s"(desc), "s"(soff) : "m0");
}
#pragma clang diagnostic pop
template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// c += w . a^T for one 16 x 16 block, in place in the accumulation registers.
// Inline assembly: where registers are left over, the compiler would give the
// builtin's result other registers than its addend and copy the accumulators
// back every step (110 -> 237 instructions per step, 82 -> 127 us at 1,024 x
// 3,072 x 12,288).  The compiler does not see it as an MFMA, so the distances
// to the vector instructions that write and read the accumulators are kept by
// hand (the s_nop before and after the K loop).
__device__ __forceinline__ void mfma16(f32x4& c, const bf16x8& w, const bf16x8& a) {
  asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(a));
}

// A tile shape: each of the 2 x 2 waves owns MB x NB blocks of 16 x 16, the X
// operand (A if XA, else W) has R ring slots and the other one R + 1.
template <int MB_, int NB_, int R_, bool XA_>
struct Shape {
  static constexpr int MB = MB_, NB = NB_, RX = R_, RY = R_ + 1;
  static constexpr bool XA = XA_;
  static constexpr int BM = 32 * MB, BN = 32 * NB;
  static constexpr int kSlotA = BM * kRowBytes, kSlotW = BN * kRowBytes;
  static constexpr int RA = XA ? RX : RY, RW = XA ? RY : RX;
  static constexpr int kBaseW = RA * kSlotA;                 // LDS: the ring of A, then the ring of W
  static constexpr int kLds = kBaseW + RW * kSlotW;
  static constexpr int LA = MB, LW = NB;                     // 1 KiB loads per wave and step
  static constexpr int LX = XA ? LA : LW, LY = XA ? LW : LA;
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
};

template <int EPI, typename S>
__global__ __launch_bounds__(kThreads, 1) void gemm_bf16_nt(
    const bf16* __restrict__ A, int64_t lda, const bf16* __restrict__ W, int64_t ldw,
    const bf16* __restrict__ bias, bf16* __restrict__ C, int64_t ldc, const bf16* R, int64_t ldr,
    const float* __restrict__ gate, int64_t gate_stride, ReqTable req, int M, int N, int K,
    int tiles_m, int tiles_n, int group_m, int plane_cols, int64_t plane_skip) {
  constexpr int MB = S::MB, NB = S::NB, BM = S::BM, BN = S::BN, RX = S::RX, RY = S::RY;
  constexpr int LA = S::LA, LW = S::LW, LX = S::LX, LY = S::LY;
  constexpr bool XA = S::XA;
  __shared__ __attribute__((aligned(1024))) char smem[S::kLds];

  const TileSeq seq = tile_seq(blockIdx.x, gridDim.x, tiles_m, tiles_n, group_m);
  if (seq.count == 0) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int KT = K / BK;

  // ---- global -> LDS.  A step's tile of an operand is pieces of 1 KiB (8
  // rows x 128 B); wave w moves pieces LA w .. LA w + LA - 1 of A and LW w ..
  // of W.  Lane i of piece q holds row 8 q + i / 8, logical chunk
  // (i % 8) ^ row_swizzle(row), and fills LDS byte 1024 q + 16 i of the slot.
  // Row 8 q + i / 8 has row_swizzle = 4 (q % 2) + i / 16, so the lane part of
  // a load's offset is one of two values per operand (by the parity of q)
  // plus a uniform number of rows; LA and LW are even, so the parity of q is
  // that of u.  A load's lane offset is its row inside the tile and its chunk,
  // the scalar offset the K step only: rows past the end of the operand (a
  // ragged last tile) read as zeros and no load leaves the operand.
  static_assert(LA % 2 == 0 && LW % 2 == 0, "the parity of a piece is that of its index in the wave");
  int a_vo[2], w_vo[2];
#pragma unroll
  for (int par = 0; par < 2; ++par) {
    const int c = (lane & 7) ^ (4 * par + (lane >> 4));
    a_vo[par] = (LA * wave * 8 + (lane >> 3)) * (int)lda * 2 + c * 16;
    w_vo[par] = (LW * wave * 8 + (lane >> 3)) * (int)ldw * 2 + c * 16;
  }
  const int a_pc = 16 * (int)lda, w_pc = 16 * (int)ldw;   // bytes of 8 rows
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  // the load cursor: step l_step of the sequence's tile l_it
  u32x4 ad{}, wd{};
  int l_it = 0, l_step = 0;
  auto set_tile = [&](int it) {
    if (it < seq.count) {
      int tm, tn;
      seq.coords(it, tm, tn);
      ad = make_desc(A + (int64_t)tm * BM * lda, ((int64_t)(M - tm * BM - 1) * lda + K) * 2);
      wd = make_desc(W + (int64_t)tn * BN * ldw, ((int64_t)(N - tn * BN - 1) * ldw + K) * 2);
    } else {   // past the last tile: empty ranges
      ad[2] = 0;
      wd[2] = 0;
    }
  };
  auto advance = [&] {
    if (++l_step == KT) {
      l_step = 0;
      set_tile(++l_it);
    }
  };
  auto load_a = [&](int u, int slot) {
    load_lds16(ad, a_vo[u & 1] + u * a_pc, l_step * (BK * 2), lds_base + slot * S::kSlotA + (LA * wave + u) * 1024);
  };
  auto load_w = [&](int u, int slot) {
    load_lds16(wd, w_vo[u & 1] + u * w_pc, l_step * (BK * 2),
               lds_base + S::kBaseW + slot * S::kSlotW + (LW * wave + u) * 1024);
  };
  auto load_x = [&](int u, int slot) { if (XA) load_a(u, slot); else load_w(u, slot); };
  auto load_y = [&](int u, int slot) { if (XA) load_w(u, slot); else load_a(u, slot); };

  // ---- fragment reads: row base + 16 b + (lane & 15), logical chunk 4 kk + (lane >> 4) of half kk
  const int fr = lane & 15, fh = lane >> 4;
  const int sw = row_swizzle(fr);   // == row_swizzle(base + 16 b + fr)
  int fo_a[2], fo_w[2];             // + 16 * kRowBytes b
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    fo_a[kk] = (wm * 16 * MB + fr) * kRowBytes + (((4 * kk + fh) ^ sw) << 4);
    fo_w[kk] = S::kBaseW + (wn * 16 * NB + fr) * kRowBytes + (((4 * kk + fh) ^ sw) << 4);
  }
  struct Frags { bf16x8 w[NB], a[MB]; };
  Frags f0, f1;
  // acc[i][j][e] = C[m][n], m = 16 MB wm + 16 j + fr and n = 16 NB wn + 16 i + 4 fh + e of the tile
  f32x4 acc[NB][MB];

  // One half: the MFMAs on f, each followed by its share of the reads of the
  // next half (half kk of the given slots) into g and of the loads, fenced so
  // that the compiler keeps this order.  The reads go first, one per 2 MFMAs,
  // so that each has half of the half to land.
  constexpr int NM = MB * NB, NR = MB + NB;
  constexpr int kReadStep = 2, kLoadStep = NM >= 48 ? 4 : 2;
  static_assert((NM - 1) / kReadStep + 1 >= NR && (NM - 1) / kLoadStep + 1 >= (LX > LY ? LX : LY), "all reads and loads are issued");
  auto half = [&](const Frags& f, Frags& g, int slot_x, int slot_y, int kk, auto loads_x, int load_slot) __attribute__((always_inline)) {
    constexpr bool kX = decltype(loads_x)::value;
    const char* const pa = smem + (XA ? slot_x : slot_y) * S::kSlotA + fo_a[kk];
    const char* const pw = smem + (XA ? slot_y : slot_x) * S::kSlotW + fo_w[kk];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const int i = m / MB, j = m % MB;
      mfma16(acc[i][j], f.w[i], f.a[j]);
      const int r = m / kReadStep;   // reads in the order of their use: w0, a0 .., w1 ..
      if (m % kReadStep == 0 && r < NR) {
        if (r == 0) g.w[0] = *reinterpret_cast<const bf16x8*>(pw);
        else if (r <= MB) g.a[r - 1] = *reinterpret_cast<const bf16x8*>(pa + (r - 1) * 16 * kRowBytes);
        else g.w[r - MB] = *reinterpret_cast<const bf16x8*>(pw + (r - MB) * 16 * kRowBytes);
      }
      const int l = m / kLoadStep;
      if (m % kLoadStep == 0 && l < (kX ? LX : LY)) {
        if (kX) load_x(l, load_slot);
        else load_y(l, load_slot);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // the first tile's steps 0 .. R - 1, then the fragments of step 0's first half
  set_tile(0);
#pragma unroll
  for (int s = 0; s < RX; ++s) {
#pragma unroll
    for (int u = 0; u < LX; ++u) load_x(u, s);
#pragma unroll
    for (int u = 0; u < LY; ++u) load_y(u, s);
    advance();
  }
  wait_vmcnt<(RX - 1) * (LX + LY)>();
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NB; ++i) f0.w[i] = *reinterpret_cast<const bf16x8*>(smem + fo_w[0] + i * 16 * kRowBytes);
#pragma unroll
  for (int j = 0; j < MB; ++j) f0.a[j] = *reinterpret_cast<const bf16x8*>(smem + fo_a[0] + j * 16 * kRowBytes);
  int sx = 0, sy = 0;   // slots of the current step, counted over all tiles: mod RX, mod RY
  for (int it = 0; it < seq.count; ++it) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{};
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");   // a vector write of an MFMA's addend
    __builtin_amdgcn_sched_barrier(0);
    int tm, tn;
    seq.coords(it, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    int last_y = 0;
    for (int s = 0; s < KT; ++s) {
      const int sx1 = sx == RX - 1 ? 0 : sx + 1;
      const int sy1 = sy == RY - 1 ? 0 : sy + 1;
      half(f0, f1, sx, sy, 1, std::false_type{}, sy == 0 ? RY - 1 : sy - 1);   // loads Y(s + R) into the slot of s - 1
      // X(s + 1) and Y(s + 1) have landed; R - 2 steps of X and R - 1 of Y may still be in flight
      wait_vmcnt<(RX - 2) * LX + (RX - 1) * LY>();
      __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
      half(f1, f0, sx1, sy1, 0, std::true_type{}, sx);                         // loads X(s + R) into the slot of s
      advance();
      last_y = sy;
      sx = sx1;
      sy = sy1;
    }
    // wait states from the last MFMA to a vector read of its result (the compiler itself would put at most 12)
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);

    // Epilogue through a wave-private LDS window of 32 rows x CW columns
    // (fp32), in the part of the last step's Y slot that this wave itself
    // refills in the next step.  Each round writes the blocks of two row
    // blocks as the MFMAs left them and reads them back row-contiguously,
    // eight columns per lane, so each global access of a wave covers whole
    // 64- or 128-byte row segments with 16 bytes per lane.  The window's 16-byte
    // chunks are permuted (even chunks of a row first) and XOR-swizzled by row
    // against bank conflicts (some are left: the conflict counter reads 0 in the
    // K loop and a fixed amount per tile, 4.4% of the LDS cycles at K = 5,120
    // and 1.8% at 13,824).  One wave's LDS
    // operations complete in order, so the window needs no barrier.  The
    // residual rows of a row block pair are loaded one pair ahead.  C may
    // alias R: every element is read before it is written, by the same lane.
    constexpr int CW = NB % 4 == 0 && LY >= 8 ? 64 : 32;   // the wave's share of a Y slot is LY KiB
    constexpr int LPR = CW / 8, RPP = 64 / LPR;            // lanes per row and rows per pass when read back
    constexpr int NP = 32 / RPP, NV = NB * 16 / CW;        // passes per window, windows per row block pair
    static_assert(32 * CW * 4 <= LY * 1024 && NB * 16 % CW == 0 && MB % 2 == 0, "the window fits");
    constexpr bool kRes = EPI == DIT_EPI_RESIDUAL || EPI == DIT_EPI_GATED_RESIDUAL;
    char* const ew = smem + (XA ? S::kBaseW + last_y * S::kSlotW : last_y * S::kSlotA) + wave * (LY * 1024);
    const int er = lane / LPR, ec = lane % LPR;
    auto at = [](int r, int c) {   // LDS byte of chunk c of window row r
      if (CW == 64) return r * 256 + ((((c >> 1) | ((c & 1) << 3)) ^ (((r & 1) << 3) | ((r >> 1) & 7))) << 4);
      return r * 128 + ((((c >> 1) | ((c & 1) << 2)) ^ ((((r >> 1) & 1) << 2) | ((r >> 2) & 3))) << 4);
    };
    const int nw = n0 + wn * 16 * NB + 8 * ec;   // the lane's first column of window 0
    float bsum[NV][8];
    int64_t c_off[NV];   // output plane of the lane's 8 columns (planes: column n in plane n / plane_cols)
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int n = nw + CW * v;
      c_off[v] = plane_cols > 0 ? (int64_t)(n / plane_cols) * plane_skip : 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) bsum[v][e] = 0.f;
      if (bias && n < N) {
        const bf16x8 bv = *reinterpret_cast<const bf16x8*>(bias + n);
#pragma unroll
        for (int e = 0; e < 8; ++e) bsum[v][e] = (float)bv[e];
      }
    }
    bf16x8 rv[2][NV][NP];
    auto load_res = [&](int j) __attribute__((always_inline)) {
      if constexpr (kRes) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            const int m = m0 + wm * 16 * MB + 32 * j + RPP * p + er, n = nw + CW * v;
            rv[j & 1][v][p] = bf16x8{};
            if (m < M && n < N) rv[j & 1][v][p] = *reinterpret_cast<const bf16x8*>(R + (int64_t)m * ldr + n);
          }
      }
    };
    load_res(0);
#pragma unroll
    for (int j = 0; j < MB / 2; ++j) {
      if (j + 1 < MB / 2) load_res(j + 1);
      const int mb = m0 + wm * 16 * MB + 32 * j;   // first row of the pair
      f32x4 gv[NV][2];
      bool g_one = true;                           // all rows of the pair belong to one request
      if (EPI == DIT_EPI_GATED_RESIDUAL) {
        const int r_lo = find_req(req.cu, req.n_req, min(mb, M - 1));
        const int r_hi = find_req(req.cu, req.n_req, min(mb + 31, M - 1));
        g_one = r_lo == r_hi;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          gv[v][0] = gv[v][1] = f32x4{};
          if (g_one && nw + CW * v < N) {
            const float* gp = gate + (int64_t)r_lo * gate_stride + nw + CW * v;
            gv[v][0] = *reinterpret_cast<const f32x4*>(gp);
            gv[v][1] = *reinterpret_cast<const f32x4*>(gp + 4);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
#pragma unroll
        for (int ii = 0; ii < CW / 16; ++ii)
#pragma unroll
          for (int jj = 0; jj < 2; ++jj)
            *reinterpret_cast<f32x4*>(ew + at(16 * jj + fr, 4 * ii + fh)) = acc[v * (CW / 16) + ii][2 * j + jj];
        const int n = nw + CW * v;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
          const int r = RPP * p + er, m = mb + r;
          const f32x4 z0 = *reinterpret_cast<const f32x4*>(ew + at(r, 2 * ec));
          const f32x4 z1 = *reinterpret_cast<const f32x4*>(ew + at(r, 2 * ec + 1));
          float z[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) z[e] = (e < 4 ? z0[e & 3] : z1[e & 3]) + bsum[v][e];
          if (EPI == DIT_EPI_GELU_TANH) {
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = gelu_tanh(z[e]);
          } else if (EPI == DIT_EPI_GATED_RESIDUAL) {
            f32x4 g0 = gv[v][0], g1 = gv[v][1];
            if (!g_one && m < M && n < N) {   // the pair spans a request boundary
              const float* gp = gate + (int64_t)find_req(req.cu, req.n_req, m) * gate_stride + n;
              g0 = *reinterpret_cast<const f32x4*>(gp);
              g1 = *reinterpret_cast<const f32x4*>(gp + 4);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = (float)rv[j & 1][v][p][e] + (e < 4 ? g0[e & 3] : g1[e & 3]) * z[e];
          } else if (EPI == DIT_EPI_RESIDUAL) {
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = (float)rv[j & 1][v][p][e] + z[e];
          }
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (bf16)z[e];
          // computed on every path: were it left to the branch, a load above
          // would be pending where the branch is not taken, and the compiler
          // would wait for all loads in the K loop (90 -> 135 us at 1,024 x
          // 3,072 x 12,288)
          asm volatile("" : "+v"(o));
          if (m < M && n < N) *reinterpret_cast<bf16x8*>(C + c_off[v] + (int64_t)m * ldc + n) = o;
        }
      }
    }
    // the window's reads are done before the next step's loads overwrite it
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
  wait_vmcnt<0>();   // no load may land in LDS after the workgroup has ended
}

// ----------------------------------------------------------------- fp32

// fp32 GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 products and
// sums).  The operands go from global memory straight into registers in the
// instruction's layout: a lane's 16-byte load holds four consecutive k of one
// row, and the four MFMAs of a 16-wide K step take element e of it, i.e. the
// same permutation of k for both operands.
//
// An output element is the sum of four partial sums over the quarters of K
// (each a multiple of 16 long), added in order, whatever the kernel:
//  - few tiles (the small exact configuration): a workgroup per 16 x 16 tile,
//    one wave per quarter, the partial sums meet in LDS.  64 x 384 outputs are
//    96 workgroups of 4 waves instead of the 6 of the former 64 x 64 FMA tiles,
//    whose one serial K loop took 47 us at K = 384 and 179 us at 1,536; now
//    4.0 and 7.3 us;
//  - else a workgroup per 64 x 64 tile, 32 x 32 per wave, the quarters one
//    after the other (a quarter of the operand reads per output).
// The small kernel reads each operand row once per 16 outputs, so its time
// grows with M N K; the line is where both take about the same time: 16.6 and
// 17.0 us at 256 x 2,048 x 512 (128 tiles of 64 x 64), 51 and 60 us at 800 x
// 512 x 2,048 (104), but 20.1 and 17.1 us at 400 x 1,536 x 512 (168).  At
// 2,048^3 the second kernel takes 236 us (73 TFLOP/s; the FMA tiles 429).
constexpr int FK = 16;   // K step
constexpr int64_t kF32LargeTiles = 128;   // 64 x 64 tiles from which the second kernel runs

// Sums over k in [k0, k1), k0 a multiple of 4, of MB x NB blocks of 16 x 16:
// acc[i][j][e] += W[n_i + 4 g + e] . A[m_j + r] with r = lane % 16, g = lane / 16.
// pa, pw: the lane's rows (k = 0), clamped to the operand's last row.
template <int MB, int NB>
__device__ __forceinline__ void f32_span(f32x4 (&acc)[NB][MB], const float* const (&pa)[MB],
                                         const float* const (&pw)[NB], int g, int k0, int k1) {
  constexpr int U = MB * NB == 1 ? 8 : 2;   // K steps in flight
  struct Step { f32x4 a[MB], w[NB]; };
  auto load = [&](Step& s, int k) {
#pragma unroll
    for (int j = 0; j < MB; ++j) s.a[j] = *reinterpret_cast<const f32x4*>(pa[j] + k + 4 * g);
#pragma unroll
    for (int i = 0; i < NB; ++i) s.w[i] = *reinterpret_cast<const f32x4*>(pw[i] + k + 4 * g);
  };
  auto mma = [&](const Step& s) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(s.w[i][e], s.a[j][e], acc[i][j], 0, 0, 0);
  };
  int k = k0;
  for (; k + FK * U <= k1; k += FK * U) {
    Step s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) load(s[u], k + FK * u);
#pragma unroll
    for (int u = 0; u < U; ++u) mma(s[u]);
  }
  if (k + FK <= k1) {   // up to U - 1 whole steps, loaded together
    Step s[U];
#pragma unroll
    for (int u = 0; u + 1 < U; ++u)
      if (k + FK * (u + 1) <= k1) load(s[u], k + FK * u);
#pragma unroll
    for (int u = 0; u + 1 < U; ++u)
      if (k + FK <= k1) {
        mma(s[u]);
        k += FK;
      }
  }
  if (k < k1) {   // the last k, one by one: a row need not be whole past k1
    Step s{};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + 4 * g + e < k1) {
#pragma unroll
        for (int j = 0; j < MB; ++j) s.a[j][e] = pa[j][k + 4 * g + e];
#pragma unroll
        for (int i = 0; i < NB; ++i) s.w[i][e] = pw[i][k + 4 * g + e];
      }
    mma(s);
  }
}

// Four output columns n .. n + 3 of row m (N is a multiple of 4, so they are all inside or all outside).
template <int EPI>
__device__ __forceinline__ void f32_store(f32x4 z, int m, int n, const float* __restrict__ bias, float* C, int64_t ldc,
                                          const float* R, int64_t ldr, const float* __restrict__ gate,
                                          int64_t gate_stride, const ReqTable& req, int M, int N, int plane_cols,
                                          int64_t plane_skip) {
  if (m >= M || n >= N) return;
  if (bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] += bias[n + e];
  }
  if (EPI == DIT_EPI_GELU_TANH) {
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = gelu_tanh(z[e]);
  }
  if (EPI == DIT_EPI_RESIDUAL || EPI == DIT_EPI_GATED_RESIDUAL) {
    const f32x4 r = *reinterpret_cast<const f32x4*>(R + (int64_t)m * ldr + n);
    if (EPI == DIT_EPI_GATED_RESIDUAL) {
      const f32x4 g4 = *reinterpret_cast<const f32x4*>(gate + (int64_t)find_req(req.cu, req.n_req, m) * gate_stride + n);
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = r[e] + g4[e] * z[e];
    } else {
      z += r;
    }
  }
  *reinterpret_cast<f32x4*>(C + (plane_cols > 0 ? (int64_t)(n / plane_cols) * plane_skip : 0) + (int64_t)m * ldc + n) = z;
}

// TILE 16: one 16 x 16 tile per workgroup, a quarter of K per wave; TILE 64:
// one 64 x 64 tile, 32 x 32 per wave.
template <int EPI, int TILE>
__global__ __launch_bounds__(256) void gemm_f32_nt(
    const float* __restrict__ A, int64_t lda, const float* __restrict__ W, int64_t ldw,
    const float* __restrict__ bias, float* C, int64_t ldc, const float* R, int64_t ldr,
    const float* __restrict__ gate, int64_t gate_stride, ReqTable req, int M, int N, int K, int plane_cols,
    int64_t plane_skip) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int kq = (K + 4 * FK - 1) / (4 * FK) * FK;   // a quarter of K
  constexpr int B = TILE == 16 ? 1 : 2;
  const int m0 = blockIdx.y * TILE + (TILE == 16 ? 0 : 32 * (wave >> 1));
  const int n0 = blockIdx.x * TILE + (TILE == 16 ? 0 : 32 * (wave & 1));
  const float *pa[B], *pw[B];
#pragma unroll
  for (int b = 0; b < B; ++b) {
    pa[b] = A + (int64_t)min(m0 + 16 * b + r, M - 1) * lda;
    pw[b] = W + (int64_t)min(n0 + 16 * b + r, N - 1) * ldw;
  }
  if constexpr (TILE == 16) {
    __shared__ f32x4 part[3][64];
    f32x4 acc[1][1] = {};
    f32_span<1, 1>(acc, pa, pw, g, min(K, wave * kq), min(K, (wave + 1) * kq));
    if (wave > 0) part[wave - 1][lane] = acc[0][0];
    __syncthreads();
    if (wave > 0) return;
    f32x4 z = acc[0][0];
#pragma unroll
    for (int q = 0; q < 3; ++q) z += part[q][lane];
    f32_store<EPI>(z, m0 + r, n0 + 4 * g, bias, C, ldc, R, ldr, gate, gate_stride, req, M, N, plane_cols, plane_skip);
  } else {
    f32x4 sum[2][2];
    for (int q = 0; q < 4; ++q) {
      f32x4 acc[2][2] = {};
      f32_span<2, 2>(acc, pa, pw, g, min(K, q * kq), min(K, (q + 1) * kq));
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) sum[i][j] = q == 0 ? acc[i][j] : sum[i][j] + acc[i][j];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        f32_store<EPI>(sum[i][j], m0 + 16 * j + r, n0 + 16 * i + 4 * g, bias, C, ldc, R, ldr, gate, gate_stride, req, M,
                       N, plane_cols, plane_skip);
  }
}

std::atomic<int> g_tile_n{0};   // forced output tile width (0: chosen per shape)

// The tile shapes, by the index of kCost.
typedef Shape<8, 8, 2, false> Tile256x256;
typedef Shape<8, 6, 2, false> Tile256x192;
typedef Shape<4, 8, 2, true> Tile128x256;
typedef Shape<4, 6, 3, false> Tile128x192;
typedef Shape<4, 4, 4, false> Tile128x128;

// What a launch of each shape takes on 256 compute units, in us: per round of
// tiles (one per compute unit) `fixed` for its start and epilogue, and per K
// step `step`, plus `full` times the share of the compute units that the round
// keeps busy (the chip slows down under load, as it runs at its power limit).
// Fitted to 98 GEMMs of the image and video blocks' projections at 100 to
// 16,000 rows, each timed with every shape and weights from the caches: the
// shape with the least estimate was the fastest one or within 1% of it in all
// of them.  With weights from memory the launches take longer than the estimate
// (at 1,024 rows up to 1.45 times), but the choice is still the fastest or
// within 2% in 30 of 32 shapes at 100 to 5,417 rows (2,048 x 9,216 x 3,072 116
// us, 109 with 256 x 192; 5,417 x 3,072 x 12,288 384, 372).  With few rows the
// small tiles use more compute units (1,024 x 3,072 x 3,072: 57 us with 256 x
// 256, 45 with 256 x 192, 24 with 128 x 128); with many rows a large tile
// reads each operand less often (16,000 x 12,288 x 3,072: 857, 895 and 1,145
// us); in between it is the rounds that decide (5,417 x 3,072 x 3,072: 124,
// 100 and 107 us, 90 with 128 x 192).
struct TileCost { int bm, bn; float fixed, step, full; };
constexpr TileCost kCost[5] = {
    {256, 256, 7.15f, 0.9445f, 0.3357f}, {256, 192, 5.97f, 0.7277f, 0.2706f}, {128, 256, 4.45f, 0.5556f, 0.1872f},
    {128, 192, 3.34f, 0.4396f, 0.1457f}, {128, 128, 2.74f, 0.3213f, 0.1101f}};

int choose_tile(int64_t M, int N, int K, int cus) {
  const int forced = g_tile_n.load(std::memory_order_relaxed);
  if (forced == 256) return 0;
  if (forced == 192) return 1;
  const float kt = (float)(K / BK);
  int best = 0;
  float least = 0.f;
  for (int t = 0; t < 5; ++t) {
    const TileCost& c = kCost[t];
    const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
    const int64_t rounds = tiles / cus, rest = tiles % cus;
    const float cost = (float)rounds * (c.fixed + kt * (c.step + c.full)) +
                       (rest ? c.fixed + kt * (c.step + c.full * (float)rest / (float)cus) : 0.f);
    if (t == 0 || cost < least) {
      best = t;
      least = cost;
    }
  }
  return best;
}

// Tile rows per raster group.  A group of G rows lets the 32 tiles resident on
// an XCD cover G x 32 / G tiles and share their panels in its L2.  Timed with
// 2, 3, 4, 6, 8 and 16 on the image and video blocks' projections at 11 to 296
// tile rows, of 128 or 256 rows as the shape was chosen: the rule is the fastest
// or within 1% of it but for a few shapes at 2 to 3% (10,240 x 5,120 x 13,824,
// 40 tile rows, 1,193 us, 1,155 with 2; 12,800 x 15,360 x 5,120, 50, 1,433, 1,390
// with 6).  9,216 x 5,120 x 5,120: 340 us with 2, 333 with 8; at 32,760 rows
// 3.51 ms with 4, 3.58 and 3.63 with 2 and 8 on the QKV shape; at 75,600 rows
// 8.29 with 3, 8.33 and 8.61 with 4 and 8.  Between 4 and 3 there is no clear
// line from 100 to 296 tile rows (1% either way).
int raster(int tiles_m) { return tiles_m <= 40 ? 8 : tiles_m <= 160 ? 4 : 3; }

template <int EPI, typename S>
hipError_t launch_tiles(const LinearArgs& p, int cus, hipStream_t s) {
  const int64_t tiles_m = (p.M + S::BM - 1) / S::BM, tiles_n = (p.N + S::BN - 1) / S::BN;
  if (tiles_m * tiles_n > 0x7FFFFFF8ll) return hipErrorInvalidValue;
  // one workgroup per compute unit, each running a sequence of tiles
  int grid = (int)((tiles_m * tiles_n + kXcds - 1) / kXcds * kXcds);
  const int resident = cus / kXcds * kXcds;
  if (resident >= kXcds && grid > resident) grid = resident;
  gemm_bf16_nt<EPI, S><<<grid, kThreads, 0, s>>>(
      (const bf16*)p.a, p.lda, (const bf16*)p.w, p.ldw, (const bf16*)p.bias, (bf16*)p.out, p.ldo,
      (const bf16*)p.res, p.ldr, p.gate, p.gate_stride, p.req, (int)p.M, p.N, p.K, (int)tiles_m, (int)tiles_n,
      raster((int)tiles_m), p.plane_cols, p.plane_stride - p.plane_cols);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_bf16(const LinearArgs& p, hipStream_t s) {
  const int cus = cu_count();
  switch (choose_tile(p.M, p.N, p.K, cus)) {
    case 0: return launch_tiles<EPI, Tile256x256>(p, cus, s);
    case 1: return launch_tiles<EPI, Tile256x192>(p, cus, s);
    case 2: return launch_tiles<EPI, Tile128x256>(p, cus, s);
    case 3: return launch_tiles<EPI, Tile128x192>(p, cus, s);
    default: return launch_tiles<EPI, Tile128x128>(p, cus, s);
  }
}

template <int EPI>
hipError_t launch_f32(const LinearArgs& p, hipStream_t s) {
  // (see gemm_f32_nt)
  const int64_t tiles = ((p.M + 63) / 64) * ((p.N + 63) / 64);
  const bool small = tiles < kF32LargeTiles;
  const int t = small ? 16 : 64;
  const dim3 grid((p.N + t - 1) / t, (unsigned)((p.M + t - 1) / t));
#define DIT_F32_ARGS                                                                                            \
  (const float*)p.a, p.lda, (const float*)p.w, p.ldw, (const float*)p.bias, (float*)p.out, p.ldo,              \
      (const float*)p.res, p.ldr, p.gate, p.gate_stride, p.req, (int)p.M, p.N, p.K, p.plane_cols,              \
      p.plane_stride - p.plane_cols
  if (small) gemm_f32_nt<EPI, 16><<<grid, 256, 0, s>>>(DIT_F32_ARGS);
  else gemm_f32_nt<EPI, 64><<<grid, 256, 0, s>>>(DIT_F32_ARGS);
#undef DIT_F32_ARGS
  return hipGetLastError();
}

}  // namespace

// Compute units of the current device (cached per device).
int cu_count() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

void set_gemm_tile_n(int bn) { g_tile_n.store(bn, std::memory_order_relaxed); }

void gemm_plan(int64_t M, int N, int K, int cus, int* tile_m, int* tile_n) {
  const TileCost& c = kCost[choose_tile(M, N, K, cus)];
  *tile_m = c.bm;
  *tile_n = c.bn;
}

hipError_t launch_linear(const LinearArgs& p, hipStream_t s) {
  if (p.M == 0) return hipSuccess;
  if (p.dtype == DIT_BF16) {
    switch (p.epi) {
      case DIT_EPI_NONE: return launch_bf16<DIT_EPI_NONE>(p, s);
      case DIT_EPI_GELU_TANH: return launch_bf16<DIT_EPI_GELU_TANH>(p, s);
      case DIT_EPI_RESIDUAL: return launch_bf16<DIT_EPI_RESIDUAL>(p, s);
      default: return launch_bf16<DIT_EPI_GATED_RESIDUAL>(p, s);
    }
  }
  switch (p.epi) {
    case DIT_EPI_NONE: return launch_f32<DIT_EPI_NONE>(p, s);
    case DIT_EPI_GELU_TANH: return launch_f32<DIT_EPI_GELU_TANH>(p, s);
    case DIT_EPI_RESIDUAL: return launch_f32<DIT_EPI_RESIDUAL>(p, s);
    default: return launch_f32<DIT_EPI_GATED_RESIDUAL>(p, s);
  }
}

}  // namespace dit
