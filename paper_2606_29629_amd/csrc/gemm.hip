// GEMMs on the matrix cores: C[M,N] = A[M,K] B[N,K]^T, bf16 operands,
// fp32 accumulation, with the layer's epilogues fused (residual add, SwiGLU,
// q/k/v split + rotary embedding + KV-cache write, fp32 store).
//
// Both operands are K-contiguous ("nn.Linear" weights [out, in] and row-major
// activations), which is the native operand layout of the bf16 MFMAs with 8
// values per lane: in v_mfma_f32_32x32x16_bf16 lane l supplies row l % 32 and
// k 8 (l / 32) .. + 7, in v_mfma_f32_16x16x32_bf16 row l % 16 and k 8 (l / 16)
// .. + 7.
//
// Tiling: BM x BN x 64 block tile, WGM x WGN waves, A and B tiles staged through
// LDS with buffer_load_dwordx4 ... lds (no register staging), 16-byte chunks
// XOR-swizzled (see swz) so that fragment reads are free of bank conflicts.
// Two main loops: the large tiles (256 x 256, 128 x 256, 128 x 128 on
// 16x16x32 MFMAs, which move half the accumulator bytes per flop through the
// register file and so hold a higher clock under the power cap) run two groups
// of waves half a phase apart, one group's reads under the other's MFMAs
// (PingLoop, PingSmall); the decode tiles (64 and 32 rows, 32x32x16) keep one
// barrier per k-tile, the loads of tile k+1 in flight while tile k computes.
//
// Dense kernel: workgroups are dispatched round-robin over the 8 XCDs; the
// linear block id is remapped so each XCD owns a contiguous range of tiles,
// walked in groups of 8 M-tiles so co-resident tiles share A and B panels in
// that XCD's L2.
//
// Grouped kernel (mixture of experts): the rows of each expert are a
// contiguous segment of the routed (permuted) order; a device-side tile table
// maps every M-tile to its expert, A rows are gathered through the
// permutation, and B is that expert's weight matrix.  The grid is sized from
// an upper bound on the tile count and surplus workgroups exit, so no count is
// read back to the host; the real tiles are dealt to the XCDs in contiguous
// shares so that an expert's M-tiles share its weights in one L2.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"

namespace tri {

constexpr int kGroupM = 8;
constexpr int kXcds = 8;
// Template-only epilogue kind: EPI_QKV with the per-head q/k RMSNorm (the
// Epi still says EPI_QKV; its q_norm pointer selects this instantiation).
constexpr int EPI_QKV_NORM = 5;

// XCD-contiguous remap of block id bid among n: the blocks of XCD x (those
// with bid % 8 == x; dispatch is round-robin over the XCDs) take one
// contiguous range of ids.
__device__ __forceinline__ int xcd_id(int bid, int n) {
  const int per = n / kXcds, rem = n % kXcds;
  const int x = bid % kXcds, loc = bid / kXcds;
  return x * per + min(x, rem) + loc;
}

// Tile of grouped-M order id: groups of kGroupM M-tiles, walked column by
// column, so co-resident tiles share A and B panels in L2.
__device__ __forceinline__ void tile_of_id(int id, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int group = id / (kGroupM * tiles_n);
  const int first_m = group * kGroupM;
  const int gm = min(kGroupM, tiles_m - first_m);
  const int in = id - group * kGroupM * tiles_n;
  tm = first_m + in % gm;
  tn = in / gm;
}

__device__ __forceinline__ void tile_of_block(int bid, int tiles_m, int tiles_n, int& tm,
                                              int& tn) {
  tile_of_id(xcd_id(bid, tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
}

// MFMA shape SH: SH x SH output blocks, KSTEP = 512 / SH of k per
// instruction, the accumulator a 16- or 4-vector per lane.
template <int SH>
struct Mfma;
template <>
struct Mfma<32> {
  using acc_t = f32x16;
  static constexpr int KSTEP = 16;
  __device__ __forceinline__ static acc_t mma(bf16x8 a, bf16x8 b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<16> {
  using acc_t = f32x4;
  static constexpr int KSTEP = 32;
  __device__ __forceinline__ static acc_t mma(bf16x8 a, bf16x8 b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// Accumulator geometry.  Block (i, j) of a wave holds C^T (the weight rows
// are the MFMA's row operand): lane l owns token row SH i + l % SH and, in
// each block, QN = SH * SH / 256 groups of four consecutive output columns,
// group q at SH j + (256 / SH) q + 4 (l / SH).  The epilogues walk the G =
// NI * QN groups of a row block: group g = QN j + q, column offset col(g)
// (plus the lane's 4 (l / SH)), values grp(acc, i, g).
//
// RH = 0: the wave's rows are contiguous, row block i at row SH i.  RH > 0
// (the ping-pong tiles): two halves of MI / 2 row blocks, RH rows apart.
template <int SH, int MI, int NI, int RH = 0>
struct AccGeo {
  using acc_t = typename Mfma<SH>::acc_t;
  static constexpr int QN = SH * SH / 256, G = NI * QN;
  __device__ __forceinline__ static constexpr int row(int i) {
    return RH ? RH * (i / (MI / 2)) + SH * (i % (MI / 2)) : SH * i;
  }
  __device__ __forceinline__ static constexpr int col(int g) {
    return SH * (g / QN) + (256 / SH) * (g % QN);
  }
  __device__ __forceinline__ static f32x4 grp(const acc_t (&acc)[MI][NI], int i, int g) {
    if constexpr (SH == 32) {
      const int j = g / 4, q = g % 4;
      return f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                   acc[i][j][4 * q + 3]};
    } else {
      return acc[i][g];
    }
  }
  __device__ __forceinline__ static int lane_row(int lane) { return lane % SH; }
  __device__ __forceinline__ static int lane_col(int lane) { return 4 * (lane / SH); }
};

// Stores of 16-bit outputs from 16 x 16 accumulator blocks.  A lane holds
// four consecutive columns of each of the groups g and g + 1 (16 columns
// apart): stored as they are, every instruction writes 32-byte pieces of 16
// rows, quarter lines that the memory side takes at ~2.5 TB/s.  One exchange
// between neighbouring 16-lane rows gives each lane eight consecutive columns
// of one group, 64-byte pieces per row: lane row lg then holds columns
// 16 (lg % 2) + 8 (lg / 2) .. + 7 of the 32, i.e. its first column moves by
// pair_shift().  (Lanes of one token row only ever exchange with each other,
// so a predicate on the row may be off for both; the exchange is its own
// inverse.)  A 4096 x 4096 output of one round of tiles: 15.3 -> 12.2 us at
// K = 64; 16384 x 37888 x 3584 3150 -> 3055 us.
__device__ __forceinline__ u32x4 pair_swap(u32x4 v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v[0], v[2], false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(v[1], v[3], false, false);
  return u32x4{a[0], b[0], a[1], b[1]};
}
__device__ __forceinline__ int pair_shift() { return 12 * ((threadIdx.x >> 4) & 1); }
__device__ __forceinline__ u32x4 pack_pair(f32x4 v0, f32x4 v1) {
  return u32x4{pack_bf16x2(v0[0], v0[1]), pack_bf16x2(v0[2], v0[3]), pack_bf16x2(v1[0], v1[1]),
               pack_bf16x2(v1[2], v1[3])};
}
// Eight columns from `col` of a row at p (wide: p + 8 columns 16-byte aligned;
// otherwise two 8-byte stores), those past N not written.
__device__ __forceinline__ void store_pair(bf16* p, u32x4 v, int col, int N, bool wide) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  if (wide && col + 8 <= N) {
    stg16(p, v);
  } else {
    if (col < N) *(u32x2*)p = u32x2{v[0], v[1]};
    if (col + 4 < N) *(u32x2*)(p + 4) = u32x2{v[2], v[3]};
  }
}

// MFMA shape of the large tiles (256 x 256, 128 x 256, 128 x 128).  The
// weight-streaming decode tiles keep 32 x 32 blocks.
constexpr int kTileSH = 16;

template <int BM, int BN, int S = 2>
struct GemmSmem {
  bf16 a[S][BM * kBK];
  bf16 b[S][BN * kBK];
};

// B-tile row -> weight row.  For SwiGLU each wave's N sub-tile holds WN/2 gate
// rows followed by the matching WN/2 up rows, so a lane owns gate and up of
// the same output column in blocks j and j + NI/2.
template <int BN, int WN>
__device__ __forceinline__ int b_row_of(int kind, int tn, int nt, int ffn) {
  if (kind == EPI_SWIGLU) {
    const int wc = nt / WN, w = nt % WN;
    const int f = tn * (BN / 2) + wc * (WN / 2) + (w % (WN / 2));
    return w < WN / 2 ? f : ffn + f;
  }
  return tn * BN + nt;
}

// Residual prefetch for the 256 x 256 residual epilogue (PingLoop).  The loads
// for the two tiles past the last one (zeros otherwise) fetch instead the two
// 128-row halves of the output tile's residual into the buffers they would
// fill: half h into buffer (KT + h) % 2, 32 rows into each half tile (A 0, A 1,
// B 0, B 1), row-major with 512-byte rows whose 16-byte chunks are stored at
// chunk ^ (row % 16) (16 consecutive rows read one logical chunk without bank
// conflicts).  Piece j of wave w in a half tile covers its rows 2 L and 2 L + 1,
// L = w + 8 j; lane l writes position l % 32 of row 2 L + l / 32, so it fetches
// logical chunk (l % 32) ^ ((2 w + l / 32) % 16) (the swizzle is an
// involution).  Rows past M, and columns past the end of row M - 1, read as zero
// through the descriptor's range.
struct ResPf {
  __amdgpu_buffer_rsrc_t rsrc;  // residual of the tile's rows (resid_range_bytes)
  uint32_t voff;                // lane part: row l / 32 of the piece, source chunk
  int ld_bytes;                 // residual row stride in bytes
  bool on;
};

// The shared K loop.  a_off / b_off: byte offset (within the buffer) of chunk
// swz(row, lane % 8) of this lane's row in each of its 1 KB LDS blocks (at or
// beyond the buffer size for rows that must read as zero).
//
// S LDS stages, tiles loaded S - 1 ahead.  Schedule of k-tile t (KSTEPS
// k-steps of one MFMA's depth): the fragments of k-step s + 1 are read from
// LDS while the MFMAs of step s run.  Before the MFMAs of the last step, each
// wave waits for its loads of tile t + 1 (those of tiles t + 2 .. t + S - 1
// may stay in flight), one barrier makes tile t + 1 visible and retires every
// read of tile t, the loads of tile t + S go into tile t's buffer and the
// first fragments of tile t + 1 are read -- all under the last step's MFMAs,
// so the barrier costs no matrix-core time beyond the skew between waves.
// Compute-bound tiles use S = 2; the decode projections, bound by the weight
// stream, use more stages for more bytes in flight per CU.
template <int BM, int BN, int WGM, int WGN, int S = 2, int SH = 32>
struct Mainloop {
  using MF = Mfma<SH>;
  using acc_t = typename MF::acc_t;
  static constexpr int NT = WGM * WGN * 64;
  static constexpr int NW = NT / 64;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int MI = WM / SH, NI = WN / SH, RH = 0;
  static constexpr int A_BLK = BM / 8 / NW, B_BLK = BN / 8 / NW;  // 1 KB blocks per wave
  static constexpr int KSTEPS = kBK / MF::KSTEP;
  static_assert(WM % SH == 0 && WN % SH == 0, "wave tile of whole MFMA blocks");

  // MA = the wave's row blocks that hold rows of the tile's valid range
  // (compile-time, MA <= MI): blocks past it would only multiply zero rows,
  // so the wave issues neither their MFMAs nor their A fragment reads (with
  // MA = 0, no MFMA and no fragment read at all).  Its share of the tile
  // loads and every barrier stay, so all waves keep the same barrier count.
  template <int MA>
  __device__ __forceinline__ static void run_rows(GemmSmem<BM, BN, S>& sm,
                                                  __amdgpu_buffer_rsrc_t ra,
                                                  const uint32_t (&a_off)[A_BLK],
                                                  __amdgpu_buffer_rsrc_t rb,
                                                  const uint32_t (&b_off)[B_BLK], int K, int wv,
                                                  int lane, acc_t (&acc)[MI][NI], int kshift) {
    static_assert(MA >= 0 && MA <= MI, "active row blocks");
    const int wm = wv / WGN, wn = wv % WGN;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = acc_t{0.f};
    // kill = 0x80000000 pushes every offset past the buffer's range, so the
    // load writes zeros instead of touching memory (used past the last tile,
    // keeping the schedule free of branches).
    // k-tile kt of the loop reads k-tile (kt + kshift) mod KT of the operands
    // (a rotation: the loop still visits every k-tile once, in a fixed order)
    const int KTr = K / kBK;
    auto kbyte = [&](int kt) {
      const int kk = kt + kshift;
      return (kk >= KTr ? kk - KTr : kk) * kBK * 2;
    };
    auto gload = [&](int kt, int buf, uint32_t kill) {
      const int kb = kbyte(kt);
#pragma unroll
      for (int j = 0; j < A_BLK; ++j)
        buffer_load_lds16(ra, &sm.a[buf][(wv + NW * j) * 8 * kBK], a_off[j] | kill, kb);
#pragma unroll
      for (int j = 0; j < B_BLK; ++j)
        buffer_load_lds16(rb, &sm.b[buf][(wv + NW * j) * 8 * kBK], b_off[j] | kill, kb);
    };
    // Fragment reads.  The lane reads row SH i + l % SH of a block and the
    // 16-byte chunk ks * KSTEP / 8 + l / SH of the step.  The swizzle of a row
    // depends on (row / 2) % 8 only, the same for rows r and r + SH i, so one
    // byte address per operand and k-step serves every block and buffer
    // (immediate offsets).
    uint32_t a_base[KSTEPS], b_base[KSTEPS];
    {
      const int lr = lane % SH, lg = lane / SH;
      const int ra0 = wm * WM + lr, rb0 = wn * WN + lr;
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        const int ch = ks * (MF::KSTEP / 8) + lg;
        a_base[ks] = (uint32_t)((ra0 * kBK + swz(ra0, ch) * 8) * 2);
        b_base[ks] = (uint32_t)((rb0 * kBK + swz(rb0, ch) * 8) * 2);
      }
    }
    const char* const lds_a = (const char*)&sm.a[0][0];
    const char* const lds_b = (const char*)&sm.b[0][0];
    auto rd_a = [&](int buf, int ks, int i) {
      return *(const bf16x8*)(lds_a + a_base[ks] + (buf * BM * kBK + i * SH * kBK) * 2);
    };
    auto rd_b = [&](int buf, int ks, int j) {
      return *(const bf16x8*)(lds_b + b_base[ks] + (buf * BN * kBK + j * SH * kBK) * 2);
    };
    bf16x8 fa[2][MI], fb[2][NI];
    auto lload = [&](int buf, int ks, int slot) {
      if constexpr (MA == 0) return;
#pragma unroll
      for (int i = 0; i < MA; ++i) fa[slot][i] = rd_a(buf, ks, i);
#pragma unroll
      for (int j = 0; j < NI; ++j) fb[slot][j] = rd_b(buf, ks, j);
    };
    // Fragment f of a k-step: f < MA -> A block f, else B block f - MA.
    auto lread = [&](int buf, int ks, int slot, int f) {
      if (f < MA) fa[slot][f] = rd_a(buf, ks, f);
      else fb[slot][f - MA] = rd_b(buf, ks, f - MA);
    };
    // Load piece p of a tile: p < A_BLK -> A block p, else B block p - A_BLK.
    auto gpiece = [&](int kt, int buf, uint32_t kill, int p) {
      const int kb = kbyte(kt);
      if (p < A_BLK)
        buffer_load_lds16(ra, &sm.a[buf][(wv + NW * p) * 8 * kBK], a_off[p] | kill, kb);
      else
        buffer_load_lds16(rb, &sm.b[buf][(wv + NW * (p - A_BLK)) * 8 * kBK],
                          b_off[p - A_BLK] | kill, kb);
    };
    // B (weight rows) as the MFMA's row operand and A (token rows) as its
    // column operand: accumulator block (i, j) holds C^T, so a lane owns one
    // token row and groups of four consecutive output columns, and the
    // epilogues move 8 or 16 contiguous bytes per lane.
    auto mfma = [&](int slot, int g) {
      const int i = g / NI, j = g % NI;
      acc[i][j] = MF::mma(fb[slot][j], fa[slot][i], acc[i][j]);
    };
    constexpr int NMF = MA * NI, NRD = MA > 0 ? MA + NI : 0, NLD = A_BLK + B_BLK;
    constexpr int NG = NMF > NRD ? NMF : NRD;
    constexpr int NGL = NG > NLD ? NG : NLD;
    const int KT = K / kBK;
    static_assert((S - 1) * NLD < 64, "vmcnt counts up to 63");
#pragma unroll
    for (int t = 0; t < S; ++t) gload(t, t, t < KT ? 0u : 0x80000000u);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * NLD) : "memory");  // tile 0 landed
    __syncthreads();
    lload(0, 0, 0);
    int buf = 0;
    // The issue order is spelled out: one MFMA, then one LDS read for the next
    // k-step (and on the last step one or more tile loads), fenced so the
    // compiler keeps it.
    auto ktile = [&](int kt) {
      const int nbuf = buf + 1 == S ? 0 : buf + 1;
#pragma unroll
      for (int ks = 0; ks + 1 < KSTEPS; ++ks) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          if (g < NMF) mfma(ks & 1, g);
          if (g < NRD) lread(buf, ks + 1, (ks + 1) & 1, g);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      constexpr int last = (KSTEPS - 1) & 1;
      // this wave's tile t + 1 loads
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * NLD) : "memory");
      __syncthreads();
      const uint32_t kill = kt + S < KT ? 0u : 0x80000000u;
#pragma unroll
      for (int g = 0; g < NGL; ++g) {
        if (g < NMF) mfma(last, g);
        if (g < NLD) gpiece(kt + S, buf, kill, g);
        if (g < NRD) lread(nbuf, 0, last ^ 1, g);  // stale but in-range on the last tile
        __builtin_amdgcn_sched_barrier(0);
      }
      buf = nbuf;
    };
    for (int kt = 0; kt < KT; ++kt) ktile(kt);
  }
  // The tile's first `rows` rows are valid: the wave runs the instantiation
  // for its active row blocks (a wave-uniform choice).
  template <int MA = MI>
  __device__ __forceinline__ static void run_valid(int rows, GemmSmem<BM, BN, S>& sm,
                                                   __amdgpu_buffer_rsrc_t ra,
                                                   const uint32_t (&a_off)[A_BLK],
                                                   __amdgpu_buffer_rsrc_t rb,
                                                   const uint32_t (&b_off)[B_BLK], int K, int wv,
                                                   int lane, acc_t (&acc)[MI][NI],
                                                   int kshift = 0) {
    const int wm = wv / WGN;
    const int act = (rows - wm * WM + SH - 1) / SH;  // row blocks holding valid rows
    if constexpr (MA == 0) {
      run_rows<0>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
    } else {
      if (act >= MA) run_rows<MA>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
      else run_valid<MA - 1>(rows, sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
    }
  }
};

// Columns of the ping-pong tiles (HB = 1 or 2: 128 HB columns, four waves
// across).  A wave's LDS rows of B are 32 wn .. + 31 of every 128-row half
// tile; b_row says which weight row each holds, so that the wave's column
// groups of 16 are its 32 HB consecutive output columns or, for SwiGLU and
// q/k/v, HB groups of one half (gate; first half of a head) and then their
// HB partners (up; second half): group g pairs with group g + HB in the same
// lane.
template <int HB>
struct PingCols {
  static constexpr int WC = 32 * HB;   // columns per wave
  // first column of wave wn, and the distance of its second HB groups
  __device__ __forceinline__ static int wave_col(int kind, int wn, int head_dim) {
    const bool qkv = kind == EPI_QKV || kind == EPI_QKV_NORM;
    const int wph = qkv ? head_dim / WC : 1;  // waves that share a head
    return (wn / wph) * wph * WC + (wn % wph) * (WC / 2);
  }
  __device__ __forceinline__ static int half_step(int kind, int head_dim) {
    return kind == EPI_QKV || kind == EPI_QKV_NORM ? head_dim / 2 : WC / 2;
  }
  __device__ __forceinline__ static int b_row(int kind, int tn, int nt, int ffn, int head_dim) {
    const int wn = (nt >> 5) & 3, g = HB == 2 ? nt >> 7 : (nt >> 4) & 1;
    const int c = HB == 2 ? nt & 31 : nt & 15;
    if (kind == EPI_SWIGLU) {
      const int f = tn * 64 * HB + wn * 16 * HB + c;
      return g ? ffn + f : f;
    }
    return tn * 128 * HB + wave_col(kind, wn, head_dim) + g * half_step(kind, head_dim) + c;
  }
};

// The 256 x 256 tiles' K loop: eight waves in two groups (waves 0-3 and 4-7,
// one of each group on every SIMD) that run the same program half a phase
// apart, so that on each SIMD one wave's MFMAs run while the other reads its
// fragments and issues its loads.
//
// A k-tile is four 16 KB half tiles (rows 0-127 and 128-255 of A and of B)
// and four phases, one per quadrant of the wave's output: wave (wm, wn) owns
// rows 64 wm .. + 63 of both A halves and rows 32 wn .. + 31 of both B halves,
// 64 x 32 per quadrant, 16 MFMAs.  Phase p of k-tile t:
//   p   reads (LDS -> registers)   loads issued            MFMAs
//   0   A0 (t)                     A1 (t + 1)              A0 B0
//   1   B1 (t)                     B0 (t + 2)              A0 B1
//   2   A1 (t)                     A0 (t + 2)              A1 B0
//   3   B0 (t + 1)                 B1 (t + 2)              A1 B1
// each phase: reads and loads, wait, barrier, MFMAs, barrier.  The second
// group passes one barrier more before the first phase (the first group one
// more at the end), which sets the groups half a phase apart.
//
// A half tile is loaded two phases or more after the phase that read its
// predecessor: that phase's reads are complete in both groups one barrier
// earlier (the second group's when its MFMAs of the phase have consumed them;
// B0, whose MFMAs come a phase later, is waited for in phase 3 itself).  It is
// read six phases after its load was issued; the wait of the phase before
// leaves the five newer half tiles' ten loads in flight.
//
// What bounds it: the board's power (gate/up at 16384 x 3584: the MFMA pipes are
// busy for 84% of the cycles, and the clock is held at 1.8 of 2.4 GHz).  A loop
// with one barrier per k-tile has to issue a k-tile's loads in one burst once
// the whole buffer is free, so a k-tile took the burst plus a memory round trip
// (3060 clocks for 2048 of MFMAs); here loads are issued at an even rate and each
// group's MFMAs cover the other's LDS reads (2450 clocks).  8192^3: 819 -> 755 us
// on random operands (1343 -> 1455 TFLOP/s), 677 -> 593 us on zeros, which draw
// less power; gate/up at 16384 x 3584 (SwiGLU) 3380 -> 3083 us, down 1720 -> 1671 us.
// Without the stagger of the groups 868 us; loads issued between the MFMAs
// 840 us; a raised wave priority around the MFMAs (8 x 2048 prefill 5950 with it,
// 5935 us without), the order of reads and loads in a phase and the order of the
// MFMAs make no difference.
struct PingLoop : PingCols<2> {
  static constexpr int SH = 16, BM = 256, BN = 256, NW = 8, NT = 512;
  using MF = Mfma<SH>;
  using acc_t = MF::acc_t;
  static constexpr int MI = 8, NI = 4;
  static constexpr int RH = 128;            // row distance of the wave's two halves
  static constexpr int A_BLK = 4, B_BLK = 4;  // 1 KB blocks per wave and k-tile
  static constexpr int KS = 2;              // 32-k steps per k-tile
  static constexpr int HALF = 128 * kBK;    // elements of a half tile

  // C0, C1: row blocks (of four) of the wave's two halves that hold valid rows.
  template <int C0, int C1, bool RPF>
  __device__ __forceinline__ static void run_rows(GemmSmem<256, 256, 2>& sm,
                                                  __amdgpu_buffer_rsrc_t ra,
                                                  const uint32_t (&a_off)[A_BLK],
                                                  __amdgpu_buffer_rsrc_t rb,
                                                  const uint32_t (&b_off)[B_BLK], int K, int wv,
                                                  int lane, acc_t (&acc)[MI][NI],
                                                  const ResPf& rp, int kshift) {
    static_assert(C0 >= 0 && C0 <= 4 && C1 >= 0 && C1 <= C0, "active row blocks");
    const int wm = wv >> 2, wn = wv & 3;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = acc_t{0.f};
    const int KT = K / kBK;
    // the two 1 KB pieces of a half tile: A (op 0) or B (op 1), half h of k-tile
    // kt; a k-tile past the last one reads zeros (kept, so that every phase
    // issues the same number of loads), or rows of the residual
    auto gload = [&](int kt, int buf, int op, int h) {
      bf16* dst = (op ? sm.b[buf] : sm.a[buf]) + h * HALF + wv * 8 * kBK;
      if (RPF && rp.on && kt >= KT) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
          buffer_load_lds16(rp.rsrc, dst + j * 64 * kBK, rp.voff,
                            (128 * (kt - KT) + 64 * op + 32 * h + 2 * (wv + 8 * j)) * rp.ld_bytes);
      } else {
        const int kk = kt + kshift;
        const int kb = (kk >= KT ? kk - KT : kk) * kBK * 2;
        const uint32_t kill = kt < KT ? 0u : 0x80000000u;
#pragma unroll
        for (int j = 0; j < 2; ++j)
          buffer_load_lds16(op ? rb : ra, dst + j * 64 * kBK,
                            (op ? b_off[2 * h + j] : a_off[2 * h + j]) | kill, kb);
      }
    };
    // fragment addresses (the swizzle of a row is that of row + 16 i)
    uint32_t a_base[KS], b_base[KS];
    {
      const int lr = lane % SH, lg = lane / SH;
      const int ra0 = wm * 64 + lr, rb0 = wn * 32 + lr;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int ch = ks * 4 + lg;
        a_base[ks] = (uint32_t)((ra0 * kBK + swz(ra0, ch) * 8) * 2);
        b_base[ks] = (uint32_t)((rb0 * kBK + swz(rb0, ch) * 8) * 2);
      }
    }
    const char* const lds_a = (const char*)&sm.a[0][0];
    const char* const lds_b = (const char*)&sm.b[0][0];
    bf16x8 fa[4][KS], fb[2][2][KS];
    auto read_a = [&](int buf, auto half) {
      constexpr int h = decltype(half)::value, C = h ? C1 : C0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < C; ++i)
          fa[i][ks] = *(const bf16x8*)(lds_a + a_base[ks] +
                                       ((buf * 2 + h) * HALF + i * SH * kBK) * 2);
    };
    auto read_b = [&](int buf, auto half) {
      constexpr int h = decltype(half)::value;
      if constexpr (C0 > 0) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            fb[h][j][ks] = *(const bf16x8*)(lds_b + b_base[ks] +
                                            ((buf * 2 + h) * HALF + j * SH * kBK) * 2);
      }
    };
    auto barrier = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    // the loads issued five phases ago have landed; then the phase's MFMAs
    // between two barriers
    auto quadrant = [&](auto ha, auto hb, bool lgkm) {
      constexpr int h = decltype(ha)::value, g = decltype(hb)::value, C = h ? C1 : C0;
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
      barrier();
      if (lgkm) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[4 * h + i][2 * g + j] = MF::mma(fb[g][j][ks], fa[i][ks], acc[4 * h + i][2 * g + j]);
      barrier();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    auto ktile = [&](int kt, auto bufc) {
      constexpr int buf = decltype(bufc)::value;
      read_a(buf, I0{});
      gload(kt + 1, buf ^ 1, 0, 1);
      quadrant(I0{}, I0{}, false);
      read_b(buf, I1{});
      gload(kt + 2, buf, 1, 0);
      quadrant(I0{}, I1{}, false);
      read_a(buf, I1{});
      gload(kt + 2, buf, 0, 0);
      quadrant(I1{}, I0{}, false);
      read_b(buf ^ 1, I0{});  // past the last tile: stale, unused
      gload(kt + 2, buf, 1, 1);
      quadrant(I1{}, I1{}, true);
    };
    gload(0, 0, 1, 0);
    gload(0, 0, 0, 0);
    gload(0, 0, 1, 1);
    gload(0, 0, 0, 1);
    gload(1, 1, 1, 0);
    gload(1, 1, 0, 0);
    gload(1, 1, 1, 1);
    asm volatile("s_waitcnt vmcnt(10)" ::: "memory");  // B0 and A0 of tile 0
    barrier();
    read_b(0, I0{});
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (wm) barrier();
    for (int kt = 0; kt < KT; kt += 2) {
      ktile(kt, I0{});
      if (kt + 1 < KT) ktile(kt + 1, I1{});
    }
    if (!wm) barrier();
    // the residual's last 32 rows (half tile A 1 of the second buffer, free
    // only now); no load may land in LDS after the workgroup's end
    if constexpr (RPF) {
      if (rp.on) gload(KT + 1, (KT + 1) & 1, 0, 1);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  // The tile's first `rows` rows are valid: each wave runs the instantiation
  // for its active row blocks, rounded up to 1, 2 or 4 of a half (a
  // wave-uniform choice; every instantiation passes the same barriers).
  template <bool RPF = false>
  __device__ __forceinline__ static void run_valid(int rows, GemmSmem<256, 256, 2>& sm,
                                                   __amdgpu_buffer_rsrc_t ra,
                                                   const uint32_t (&a_off)[A_BLK],
                                                   __amdgpu_buffer_rsrc_t rb,
                                                   const uint32_t (&b_off)[B_BLK], int K, int wv,
                                                   int lane, acc_t (&acc)[MI][NI],
                                                   int kshift = 0, const ResPf& rp = ResPf{}) {
    const int wm = wv >> 2;
    const int c0 = (rows - wm * 64 + SH - 1) / SH;        // blocks of the first half
    const int c1 = (rows - 128 - wm * 64 + SH - 1) / SH;  // of the second
    if (c1 > 2) run_rows<4, 4, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
    else if (c1 > 1) run_rows<4, 2, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
    else if (c1 > 0) run_rows<4, 1, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
    else if (c0 > 2) run_rows<4, 0, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
    else if (c0 > 1) run_rows<2, 0, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
    else if (c0 > 0) run_rows<1, 0, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
    else run_rows<0, 0, RPF>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, rp, kshift);
  }

};

// The same staggered scheme for 128-row tiles of 128 HB columns (HB = 1, 2):
// a wave owns 64 x 32 HB outputs, HB phases of 16 MFMAs per k-tile.
//   HB = 2, three stages:  phase 0 reads A, B0 (t), loads B1 (t + 2)
//                          phase 1 reads B1 (t), loads A, B0 (t + 3)
//   HB = 1, five stages:   reads A, B (t), loads A, B (t + 4)
// A phase's reads are waited for before its first barrier, so a stage is
// loaded again from the next phase on: the four (three) youngest phases'
// loads, up to 96 KB per CU, stay in flight.
// What bounds it: one k-tile's loads (32 or 48 KB) take as long from L2 as its
// MFMAs (ragged prefill of 1061 tokens: waves wait for 34 to 44% of their cycles,
// 4 to 6% on LDS).  The four- and eight-wave loops with one barrier per k-tile that
// these replace waited for LDS and for each load burst instead.
template <int HB>
struct PingSmall : PingCols<HB> {
  static constexpr int SH = 16, BM = 128, BN = 128 * HB, NW = 8, NT = 512;
  static constexpr int S = HB == 1 ? 5 : 3;
  using MF = Mfma<SH>;
  using acc_t = MF::acc_t;
  using Smem = GemmSmem<BM, BN, S>;
  static constexpr int MI = 4, NI = 2 * HB, RH = 0;
  static constexpr int A_BLK = 2, B_BLK = 2 * HB;
  static constexpr int KS = 2;

  template <int C>
  __device__ __forceinline__ static void run_rows(Smem& sm, __amdgpu_buffer_rsrc_t ra,
                                                  const uint32_t (&a_off)[A_BLK],
                                                  __amdgpu_buffer_rsrc_t rb,
                                                  const uint32_t (&b_off)[B_BLK], int K, int wv,
                                                  int lane, acc_t (&acc)[MI][NI], int kshift) {
    const int wm = wv >> 2, wn = wv & 3;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = acc_t{0.f};
    const int KT = K / kBK;
    // k-tile kt's A (op 0) or half h of B (op 1): two 1 KB pieces per wave; past
    // the last k-tile zeros, so that every phase issues the same loads
    auto gload = [&](int kt, int op, int h) {
      const int st = kt % S;
      bf16* dst = (op ? sm.b[st] : sm.a[st]) + h * 128 * kBK + wv * 8 * kBK;
      const int kk = kt + kshift;
      const int kb = (kk >= KT ? kk - KT : kk) * kBK * 2;
      const uint32_t kill = kt < KT ? 0u : 0x80000000u;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        buffer_load_lds16(op ? rb : ra, dst + j * 64 * kBK, (op ? b_off[2 * h + j] : a_off[j]) | kill,
                          kb);
    };
    uint32_t a_base[KS], b_base[KS];
    {
      const int lr = lane % SH, lg = lane / SH;
      const int ra0 = wm * 64 + lr, rb0 = wn * 32 + lr;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int ch = ks * 4 + lg;
        a_base[ks] = (uint32_t)((ra0 * kBK + swz(ra0, ch) * 8) * 2);
        b_base[ks] = (uint32_t)((rb0 * kBK + swz(rb0, ch) * 8) * 2);
      }
    }
    bf16x8 fa[4][KS], fb[HB][2][KS];
    auto read_a = [&](int st) {
      const char* p = (const char*)sm.a[st];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < C; ++i) fa[i][ks] = *(const bf16x8*)(p + a_base[ks] + i * SH * kBK * 2);
    };
    auto read_b = [&](int st, auto half) {
      constexpr int h = decltype(half)::value;
      const char* p = (const char*)(sm.b[st] + h * 128 * kBK);
      if constexpr (C > 0) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            fb[h][j][ks] = *(const bf16x8*)(p + b_base[ks] + j * SH * kBK * 2);
      }
    };
    auto barrier = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    // 12 loads stay in flight either way: HB = 1, the three youngest k-tiles;
    // HB = 2, the loads of the four youngest phases
    auto phase = [&](auto half) {
      constexpr int h = decltype(half)::value;
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
      barrier();
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][2 * h + j] = MF::mma(fb[h][j][ks], fa[i][ks], acc[i][2 * h + j]);
      barrier();
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, HB - 1>;
    if constexpr (HB == 1) {
      for (int t = 0; t < S - 1; ++t) {
        gload(t, 0, 0);
        gload(t, 1, 0);
      }
    } else {
      gload(0, 0, 0);
      gload(0, 1, 0);
      gload(0, 1, 1);
      gload(1, 0, 0);
      gload(1, 1, 0);
      gload(1, 1, 1);
      gload(2, 0, 0);
      gload(2, 1, 0);
    }
    asm volatile("s_waitcnt vmcnt(12)" ::: "memory");  // the first phase's tiles
    barrier();
    if (wm) barrier();
    int st = 0;
    for (int kt = 0; kt < KT; ++kt) {
      read_a(st);
      read_b(st, I0{});
      if constexpr (HB == 1) {
        gload(kt + S - 1, 0, 0);
        gload(kt + S - 1, 1, 0);
        phase(I0{});
      } else {
        gload(kt + 2, 1, 1);
        phase(I0{});
        read_b(st, I1{});
        gload(kt + 3, 0, 0);
        gload(kt + 3, 1, 0);
        phase(I1{});
      }
      st = st + 1 == S ? 0 : st + 1;
    }
    if (!wm) barrier();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may land after the end
  }
  __device__ __forceinline__ static void run_valid(int rows, Smem& sm, __amdgpu_buffer_rsrc_t ra,
                                                   const uint32_t (&a_off)[A_BLK],
                                                   __amdgpu_buffer_rsrc_t rb,
                                                   const uint32_t (&b_off)[B_BLK], int K, int wv,
                                                   int lane, acc_t (&acc)[MI][NI],
                                                   int kshift = 0) {
    const int c = (rows - (wv >> 2) * 64 + SH - 1) / SH;
    if (c > 2) run_rows<4>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
    else if (c > 1) run_rows<2>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
    else if (c > 0) run_rows<1>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
    else run_rows<0>(sm, ra, a_off, rb, b_off, K, wv, lane, acc, kshift);
  }
};

// Main loop of a tile form: 2 x 4 waves on 16 x 16 blocks are the ping-pong
// forms (256 x 256, 128 x 256, 128 x 128).
template <int BM, int BN, int WGM, int WGN, int S, int SH>
constexpr bool is_ping() {
  return WGM == 2 && WGN == 4 && SH == 16;
}
template <int BM, int BN, int WGM, int WGN, int S, int SH>
using MainloopOf = std::conditional_t<
    is_ping<BM, BN, WGM, WGN, S, SH>(),
    std::conditional_t<BM == 256, PingLoop, PingSmall<BN / 128>>, Mainloop<BM, BN, WGM, WGN, S, SH>>;

// Epilogues.  The accumulators are read by column group (AccGeo): row0 =
// output row of the lane in row block 0 (including l % SH); col0 = output
// column of the lane's first group (including 4 (l / SH)).  Rows >= row_lim
// and column groups >= N are not written (N is a multiple of 4).  Operands
// of a lane's row (residual) are loaded for a whole row block before any
// store, at clamped addresses, so no load waits behind a store.
// The second half of a wave's column groups starts hs columns after the first
// (half the wave's columns, unless the tile deals a head's halves apart).
template <int SH, int MI, int NI, int EK, int RH = 0>
__device__ __forceinline__ void plain_epilogue(
    const typename Mfma<SH>::acc_t (&acc)[MI][NI], const Epi& epi, int row0, int row_lim,
    int col0, int N, int hs = NI * SH / 2) {
  using Geo = AccGeo<SH, MI, NI, RH>;
  constexpr int G = Geo::G;
  auto gcol = [&](int g) { return g < G / 2 ? Geo::col(g) : Geo::col(g - G / 2) + hs; };
  constexpr int KIND = EK & kEpiKindMask;
  using T = typename Store<(EK & kEpiF32) != 0>::T;
  typedef T T4 __attribute__((ext_vector_type(4)));
  const T* __restrict__ resid = (const T*)epi.resid;
  if constexpr (SH == 16 && sizeof(T) == 2 && KIND != EPI_STORE_F32) {
    // pairs of groups within a half (of two groups, the halves are adjacent)
    static_assert(G % 4 == 0 || G == 2, "whole pairs");
    const bool wide = (epi.ldo & 7) == 0 && (KIND != EPI_RESID || (epi.ldr & 7) == 0);
    const int c0 = col0 + pair_shift();
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int row = row0 + Geo::row(i);
      const int rc = min(row, row_lim - 1);
      u32x4 res[G / 2];
      if constexpr (KIND == EPI_RESID) {
        // (clamped: groups of four columns, N is a multiple of 4)
        const T* rp = resid + (int64_t)rc * epi.ldr;
#pragma unroll
        for (int q = 0; q < G / 2; ++q) {
          const int col = c0 + gcol(2 * q);
          if (wide) {
            res[q] = ldg16(rp + min(col, N - 8));
          } else {
            const u32x2 a = *(const u32x2*)(rp + min(col, N - 4));
            const u32x2 b = *(const u32x2*)(rp + min(col + 4, N - 4));
            res[q] = u32x4{a[0], a[1], b[0], b[1]};
          }
        }
      }
      if (row >= row_lim) continue;
#pragma unroll
      for (int q = 0; q < G / 2; ++q) {
        f32x4 v0 = Geo::grp(acc, i, 2 * q), v1 = Geo::grp(acc, i, 2 * q + 1);
        if constexpr (KIND == EPI_RESID) {
          Pack8 r;
          r.u = pair_swap(res[q]);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v0[e] += bf2f(r.e[e]);
            v1[e] += bf2f(r.e[4 + e]);
          }
        }
        const int col = c0 + gcol(2 * q);
        store_pair((bf16*)epi.out + (int64_t)row * epi.ldo + col, pair_swap(pack_pair(v0, v1)), col,
                   N, wide);
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int row = row0 + Geo::row(i);
    const int rc = min(row, row_lim - 1);
    T4 res[G];
    if constexpr (KIND == EPI_RESID) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int col = min(col0 + gcol(g), N - 4);
        res[g] = *(const T4*)(resid + (int64_t)rc * epi.ldr + col);
      }
    }
    if (row >= row_lim) continue;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int col = col0 + gcol(g);
      if (col >= N) continue;
      const f32x4 v = Geo::grp(acc, i, g);
      if constexpr (KIND == EPI_STORE_F32) {
        *(f32x4*)((float*)epi.out + (int64_t)row * epi.ldo + col) = v;
      } else {
        T4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x = v[e];
          if constexpr (KIND == EPI_RESID) x += (float)res[g][e];
          o[e] = (T)x;
        }
        *(T4*)((T*)epi.out + (int64_t)row * epi.ldo + col) = o;
      }
    }
  }
}

// The residual epilogue of a 256 x 256 tile whose residual was prefetched
// into LDS (ResPf): tile-relative row tr / column tc of the lane's first group
// (row0 - tile row0 and col0 - tile col0), kt_par = KT % 2.  The caller has
// waited for the prefetch loads and passed a barrier.
template <int SH, int MI, int NI, int RH>
__device__ __forceinline__ void resid_lds_epilogue(
    const typename Mfma<SH>::acc_t (&acc)[MI][NI], const Epi& epi, int row0, int row_lim,
    int col0, int N, const char* smem, int kt_par, int tr, int tc) {
  using Geo = AccGeo<SH, MI, NI, RH>;
  constexpr int G = Geo::G;
  constexpr int kRegion = 128 * kBK * 2;  // bytes of one half tile
  const bool wide = (epi.ldo & 7) == 0;
  typedef bf16 T4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int row = row0 + Geo::row(i), r = tr + Geo::row(i);
    const int h = r >> 7, reg = (r >> 5) & 3, rr = r & 31;
    // half tile reg of the buffer: A halves 0 and 1, then (past both A
    // buffers) B halves 0 and 1
    const char* rbase = smem + (reg >> 1) * 4 * kRegion + ((kt_par + h) & 1) * 2 * kRegion +
                        (reg & 1) * kRegion + rr * 512;
    T4 res[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int c = tc + Geo::col(g);
      res[g] = *(const T4*)(rbase + (((c >> 3) ^ (rr & 15)) << 4) + (c & 7) * 2);
    }
    if (row >= row_lim) continue;
#pragma unroll
    for (int q = 0; q < G / 2; ++q) {
      f32x4 v0 = Geo::grp(acc, i, 2 * q), v1 = Geo::grp(acc, i, 2 * q + 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v0[e] += (float)res[2 * q][e];
        v1[e] += (float)res[2 * q + 1][e];
      }
      const int col = col0 + pair_shift() + Geo::col(2 * q);
      store_pair((bf16*)epi.out + (int64_t)row * epi.ldo + col, pair_swap(pack_pair(v0, v1)), col,
                 N, wide);
    }
  }
}

// SwiGLU: the first half of a wave's columns holds gate rows, the second half
// the matching up rows (b_row_of), so group g < G / 2 pairs with g + G / 2;
// f0 = output column (intermediate index) of the lane's first group.
template <int SH, int MI, int NI, bool F32, int RH = 0>
__device__ __forceinline__ void swiglu_epilogue(const typename Mfma<SH>::acc_t (&acc)[MI][NI],
                                                const Epi& epi, int row0, int row_lim, int f0) {
  using Geo = AccGeo<SH, MI, NI, RH>;
  constexpr int G = Geo::G;
  using T = typename Store<F32>::T;
  typedef T T4 __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int row = row0 + Geo::row(i);
    if (row >= row_lim) continue;
    if constexpr (SH == 16 && !F32 && G >= 4) {
      // (ffn is a multiple of 64: whole pairs of groups, 16-byte stores)
#pragma unroll
      for (int q = 0; q < G / 4; ++q) {
        f32x4 o[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const f32x4 gt = Geo::grp(acc, i, 2 * q + u), up = Geo::grp(acc, i, 2 * q + u + G / 2);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[u][e] = silu(gt[e]) * up[e];
        }
        const int f = f0 + pair_shift() + Geo::col(2 * q);
        const u32x4 v = pair_swap(pack_pair(o[0], o[1]));
        if (f < epi.ffn) stg16((bf16*)epi.out + (int64_t)row * epi.ldo + f, v);
      }
      continue;
    }
#pragma unroll
    for (int g = 0; g < G / 2; ++g) {
      const int f = f0 + Geo::col(g);
      if (f >= epi.ffn) continue;
      const f32x4 gt = Geo::grp(acc, i, g), up = Geo::grp(acc, i, g + G / 2);
      T4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (T)(silu(gt[e]) * up[e]);
      *(T4*)((T*)epi.out + (int64_t)row * epi.ldo + f) = o;
    }
  }
}

// QB consecutive first-half groups g0 .. g0 + QB - 1 of row block i, all in
// one q (KIND 0), k (1) or v (2) head: the lane's token row, head-dim values
// d + (col(g0 + u) - col(g0)) + e of the first half and the same plus D / 2
// from group g0 + u + GH.  NRM: the values are normalised and have their bias.
template <int KIND, int SH, int MI, int NI, int GH, int QB, bool F32, int RH = 0, bool NRM = false>
__device__ __forceinline__ void qkv_block(const typename Mfma<SH>::acc_t (&acc)[MI][NI],
                                          const Epi& epi, int i, int g0, int D, int row0, int M,
                                          int head, int d, const float (&b1)[QB][4],
                                          const float (&b2)[QB][4]) {
  using Geo = AccGeo<SH, MI, NI, RH>;
  const int half = D / 2;
  using T = typename Store<F32>::T;
  typedef T T4 __attribute__((ext_vector_type(4)));
  const int Hq = epi.n_q_heads, Hkv = epi.n_kv_heads;
  const int row = row0 + Geo::row(i);
  const int rc = min(row, M - 1);
  f32x4 cs[QB][2];  // (cos, sin) of the group's 4 values: [u][0] = e 0..1, [u][1] = e 2..3
  int sl = 0, tr = 0;
  if constexpr (KIND != 2) {
    const float2* __restrict__ rp = epi.rope + (int64_t)rc * half + d;
#pragma unroll
    for (int u = 0; u < QB; ++u) {
      const int dc = Geo::col(g0 + u) - Geo::col(g0);
      cs[u][0] = *(const f32x4*)(rp + dc);
      cs[u][1] = *(const f32x4*)(rp + dc + 2);
    }
  }
  if constexpr (KIND != 0) {
    sl = epi.tok_slot[rc];
    tr = epi.tok_row[rc];
  }
  if (row >= M) return;
  T* p;
  if constexpr (KIND == 0) {
    p = (T*)epi.q + ((int64_t)row * Hq + head) * D + d;
  } else {
    if (sl < 0) return;
    const int kvh = KIND == 1 ? head - Hq : head - Hq - Hkv;
    p = (T*)(KIND == 1 ? epi.kc : epi.vc) + (((int64_t)sl * Hkv + kvh) * epi.max_seq + tr) * D + d;
  }
  f32x4 o1[QB], o2[QB];
#pragma unroll
  for (int u = 0; u < QB; ++u) {
    const f32x4 v1 = Geo::grp(acc, i, g0 + u), v2 = Geo::grp(acc, i, g0 + u + GH);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x1 = NRM ? v1[e] : v1[e] + b1[u][e], x2 = NRM ? v2[e] : v2[e] + b2[u][e];
      if constexpr (KIND != 2) {
        const float c = cs[u][e >> 1][2 * (e & 1)], sn = cs[u][e >> 1][2 * (e & 1) + 1];
        // (the fused multiply-adds are written out: which product of a sum is
        // rounded is otherwise the compiler's choice in each instantiation)
        const float y1 = fmaf(x1, c, -(x2 * sn));
        const float y2 = NRM ? fmaf(x2, c, x1 * sn) : fmaf(x1, sn, x2 * c);
        x1 = y1;
        x2 = y2;
      }
      o1[u][e] = x1;
      o2[u][e] = x2;
    }
  }
  if constexpr (SH == 16 && !F32 && QB % 2 == 0) {
    T* const ps = p + pair_shift();
#pragma unroll
    for (int u = 0; u < QB; u += 2) {
      const int dc = Geo::col(g0 + u) - Geo::col(g0);
      stg16(ps + dc, pair_swap(pack_pair(o1[u], o1[u + 1])));
      stg16(ps + dc + half, pair_swap(pack_pair(o2[u], o2[u + 1])));
    }
  } else {
#pragma unroll
    for (int u = 0; u < QB; ++u) {
      const int dc = Geo::col(g0 + u) - Geo::col(g0);
      T4 s1, s2;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s1[e] = (T)o1[u][e];
        s2[e] = (T)o2[u][e];
      }
      *(T4*)(p + dc) = s1;
      *(T4*)(p + dc + half) = s2;
    }
  }
}

// The q/k/v epilogue of the ping-pong tiles: the wave's first HB column groups
// are first-half values of one head, the others their rotary partners
// (PingCols).  NORM: the per-head RMSNorm of q and k; a lane and the three
// others of its row hold 32 HB of the head's values, the rest are the
// neighbour waves', whose sums of squares come through LDS (free past the
// main loop), as do the gains.
struct QkvNormSmem {
  float ss[8][128];   // [wave][row of the wave]
  float gain[2][128];  // q, k
};

template <class ML, int KIND, bool NORM, bool F32>
__device__ __forceinline__ void qkv_ping_rows(typename ML::acc_t (&acc)[ML::MI][ML::NI],
                                              const Epi& epi, const QkvNormSmem& sm, int wv,
                                              int row0, int M, int head, int d,
                                              const float (&b1)[ML::NI / 2][4],
                                              const float (&b2)[ML::NI / 2][4]) {
  constexpr int SH = 16, MI = ML::MI, NI = ML::NI, HB = NI / 2, RH = ML::RH;
  constexpr bool NRM = NORM && KIND != 2;
  const int D = epi.head_dim, lr = threadIdx.x & 15;
  const int wph = D / ML::WC;  // waves that share a head: 1, 2 or 4
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if constexpr (NRM) {
      const float(*sp)[128] = &sm.ss[wv / wph * wph];
      float ss = sp[0][16 * i + lr];
      if (wph > 1) ss += sp[1][16 * i + lr];
      if (wph > 2) ss += sp[2][16 * i + lr] + sp[3][16 * i + lr];
      const float r = 1.0f / sqrtf(ss / (float)D + epi.eps);
      // (the bias is added here, and not again below)
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        const f32x4 g1 = *(const f32x4*)&sm.gain[KIND][d + 16 * u];
        const f32x4 g2 = *(const f32x4*)&sm.gain[KIND][d + 16 * u + D / 2];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[i][u][e] = (acc[i][u][e] + b1[u][e]) * (r * g1[e]);
          acc[i][u + HB][e] = (acc[i][u + HB][e] + b2[u][e]) * (r * g2[e]);
        }
      }
      qkv_block<KIND, SH, MI, NI, HB, HB, F32, RH, true>(acc, epi, i, 0, D, row0, M, head, d, b1, b2);
    } else {
      qkv_block<KIND, SH, MI, NI, HB, HB, F32, RH>(acc, epi, i, 0, D, row0, M, head, d, b1, b2);
    }
    if constexpr (NORM) __builtin_amdgcn_sched_barrier(0);  // one row block at a time: no spills
  }
}

template <class ML, bool NORM, bool F32>
__device__ __forceinline__ void qkv_ping_epilogue(typename ML::acc_t (&acc)[ML::MI][ML::NI],
                                                  const Epi& epi, char* smem, int wv, int lane,
                                                  int tile_row, int tile_col, int M, int N) {
  using St = Store<F32>;
  constexpr int MI = ML::MI, HB = ML::NI / 2;
  const int wm = wv >> 2, wn = wv & 3;
  const int lr = lane & 15, lc = 4 * (lane >> 4);
  const int D = epi.head_dim, half = D / 2, Hq = epi.n_q_heads, Hkv = epi.n_kv_heads;
  const int wcol = tile_col + ML::wave_col(EPI_QKV, wn, D);
  const bool live = wcol < N;  // wave-uniform (whole heads: N is a multiple of D)
  const int col = (live ? wcol : 0) + lc;
  const int head = col / D, d = col % D;
  const int kind = __builtin_amdgcn_readfirstlane(head < Hq ? 0 : (head < Hq + Hkv ? 1 : 2));
  const int row0 = tile_row + wm * 64 + lr;
  QkvNormSmem& sm = *reinterpret_cast<QkvNormSmem*>(smem);
  float b1[HB][4], b2[HB][4];
#pragma unroll
  for (int u = 0; u < HB; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      b1[u][e] = epi.bias ? St::ld(epi.bias, col + 16 * u + e) : 0.f;
      b2[u][e] = epi.bias ? St::ld(epi.bias, col + 16 * u + e + half) : 0.f;
    }
  if constexpr (NORM) {
    __syncthreads();  // every wave is done with the main loop's LDS
    if (threadIdx.x < 256) {
      const int w = threadIdx.x >> 7, c = threadIdx.x & 127;
      if (c < D) sm.gain[w][c] = St::ld(w ? epi.k_norm : epi.q_norm, c);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      // by four columns, then lanes, then groups (waves below): a tree that is
      // the same for every tile form
      float su[HB];
#pragma unroll
      for (int u = 0; u < HB; ++u) {
        su[u] = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x1 = acc[i][u][e] + b1[u][e], x2 = acc[i][u + HB][e] + b2[u][e];
          su[u] += x1 * x1 + x2 * x2;
        }
        su[u] += __shfl_xor(su[u], 16, 64);
        su[u] += __shfl_xor(su[u], 32, 64);
      }
      static_assert(HB == 1 || HB == 2, "a wave's first-half groups of a head");
      const float ss = HB == 2 ? su[0] + su[HB - 1] : su[0];
      if (lane < 16) sm.ss[wv][16 * i + lr] = ss;
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // (the biased sums are formed again below: kept from here, they would spill)
#pragma unroll
    for (int u = 0; u < HB; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) asm("" : "+v"(b1[u][e]), "+v"(b2[u][e]));
  }
  if (!live) return;
  if (kind == 0) qkv_ping_rows<ML, 0, NORM, F32>(acc, epi, sm, wv, row0, M, head, d, b1, b2);
  else if (kind == 1) qkv_ping_rows<ML, 1, NORM, F32>(acc, epi, sm, wv, row0, M, head, d, b1, b2);
  else qkv_ping_rows<ML, 2, NORM, F32>(acc, epi, sm, wv, row0, M, head, d, b1, b2);
}

template <int BM, int BN, int WGM, int WGN, int EK, int S = 2, int SH = 32>
__global__ __launch_bounds__(WGM * WGN * 64, 1) void gemm_kernel(const bf16* __restrict__ A, int lda,
                                                   const bf16* __restrict__ B, int ldb, int M,
                                                   int N, int K, int kc, Epi epi,
                                                   int tiles_m, int tiles_n, int full,
                                                   int tsplit, float* __restrict__ tail) {
  using ML = MainloopOf<BM, BN, WGM, WGN, S, SH>;
  constexpr bool PP = is_ping<BM, BN, WGM, WGN, S, SH>();
  constexpr int RH = ML::RH;
  using Geo = AccGeo<SH, ML::MI, ML::NI, RH>;
  constexpr int NW = ML::NW, MI = ML::MI, NI = ML::NI;
  constexpr int WM = PP ? 64 : BM / WGM, WN = BN / WGN;
  constexpr int KIND = EK & kEpiKindMask;
  constexpr bool F32 = (EK & kEpiF32) != 0;
  extern __shared__ __align__(16) char smem_raw[];
  GemmSmem<BM, BN, S>& sm = *reinterpret_cast<GemmSmem<BM, BN, S>*>(smem_raw);

  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / WGN, wn = wv % WGN;
  // Blocks [0, full) run whole tiles (ids 0 .. full-1 of the grouped order);
  // the ones after it run the last tiles in `tsplit` K-splits each (fp32
  // partials to `tail`), so that a final partial round fills every CU.
  // Half-tile mode (tsplit == 0, 128-row tiles): the grid covers the last
  // tiles of a 256-row grid (tiles_m of 256 rows, ids from `full`) as two
  // 128-row halves each, over the whole K; the two halves of a tile are
  // consecutive ids, so the XCD remap keeps them in one L2.
  int tm, tn, u = -1;
  if (BM == 128 && tsplit == 0) {
    const int id = xcd_id(blockIdx.x, (int)gridDim.x);
    tile_of_id(full + id / 2, tiles_m, tiles_n, tm, tn);
    tm = 2 * tm + (id & 1);
    if (tm * BM >= M) return;  // the empty half of a last M-tile
  } else if ((int)blockIdx.x < full) {
    tile_of_id(xcd_id(blockIdx.x, full), tiles_m, tiles_n, tm, tn);
  } else {
    u = blockIdx.x - full;
    tile_of_id(full + u / tsplit, tiles_m, tiles_n, tm, tn);
    kc = cdiv(K / kBK, tsplit) * kBK;  // the last split takes the remainder
  }
  const int n_rows_b = KIND == EPI_SWIGLU ? 2 * epi.ffn : N;
  // Split-K (fp32 partial output only): split z covers k in [z kc, z kc + kc)
  // and writes plane z of the output.
  const int k0 = (u >= 0 ? u % tsplit : (int)blockIdx.y) * kc;
  K = min(kc, K - k0);
  A += k0;
  B += k0;

  // Buffer descriptors: rows past the end of A or B read as zero.
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
      (void*)A, (short)0, (int)((int64_t)M * lda * 2 - (int64_t)k0 * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
      (void*)B, (short)0, (int)((int64_t)n_rows_b * ldb * 2 - (int64_t)k0 * 2), 0x00020000);
  // Global -> LDS without registers: each buffer_load_dwordx4 ... lds writes the
  // 64 lanes' 16 bytes to 1 KB of LDS in lane order, i.e. 8 tile rows.  Lane l
  // fills physical chunk l % 8 of row 8 b + l / 8 of its block b, so it fetches
  // the logical chunk swz(row, l % 8) of that row (swz is an involution).
  const int lrow = lane >> 3;
  uint32_t a_off[ML::A_BLK], b_off[ML::B_BLK];
#pragma unroll
  for (int j = 0; j < ML::A_BLK; ++j) {
    const int tr = (wv + NW * j) * 8 + lrow;  // tile row
    const int gr = tm * BM + tr;
    a_off[j] = gr < M ? (uint32_t)(((int64_t)gr * lda + swz(tr, lane & 7) * 8) * 2) : 0x80000000u;
  }
#pragma unroll
  for (int j = 0; j < ML::B_BLK; ++j) {
    const int tr = (wv + NW * j) * 8 + lrow;
    int gr;
    if constexpr (PP) gr = ML::b_row(KIND, tn, tr, epi.ffn, epi.head_dim);
    else gr = b_row_of<BN, WN>(KIND, tn, tr, epi.ffn);
    b_off[j] = gr < n_rows_b ? (uint32_t)(((int64_t)gr * ldb + swz(tr, lane & 7) * 8) * 2) : 0x80000000u;
  }
  typename ML::acc_t acc[MI][NI];
  const int lr = Geo::lane_row(lane), lc = Geo::lane_col(lane);
  // bf16 residual epilogue of a whole 256 x 256 tile: prefetch the residual
  // into the LDS buffers freed by the last two k-tiles (ResPf)
  constexpr bool kResPf = KIND == EPI_RESID && !F32 && PP && BM == 256;
  // The descriptor is built unconditionally (only `on` depends on the split):
  // a descriptor assigned under a run-time branch ends up in private memory,
  // and a kernel with a private segment slows every later dispatch on its
  // queue.
  ResPf rp{};
  if constexpr (kResPf) {
    const int ld_bytes = epi.ldr * 2;
    rp = ResPf{__builtin_amdgcn_make_buffer_rsrc(
                   (void*)((const bf16*)epi.resid + (int64_t)tm * BM * epi.ldr + tn * BN),
                   (short)0, resid_range_bytes(M, epi.ldr, tm * BM, tn * BN, BM), 0x00020000),
               (uint32_t)((lane >> 5) * ld_bytes +
                          (((lane & 31) ^ ((2 * wv + (lane >> 5)) & 15)) << 4)),
               ld_bytes, u < 0 && K / kBK >= 2};
  }
  if constexpr (PP && BM == 256)
    ML::template run_valid<kResPf>(M - tm * BM, sm, rsrc_a, a_off, rsrc_b, b_off, K, wv, lane, acc,
                                   0, rp);
  else
    ML::run_valid(M - tm * BM, sm, rsrc_a, a_off, rsrc_b, b_off, K, wv, lane, acc);
  // the wave's first column within the tile, and its second half's distance
  int wcol = wn * WN, hs = WN / 2;
  if constexpr (PP) {
    wcol = ML::wave_col(KIND, wn, epi.head_dim);
    hs = ML::half_step(KIND, epi.head_dim);
  }

  if (u >= 0) {  // tail split: the tile's fp32 partial sums, [BM][BN]
    Epi e{};
    e.out = tail + (int64_t)u * BM * BN;
    e.ldo = BN;
    // (the tile's valid rows only: tail_epi_kernel reads no others)
    plain_epilogue<SH, MI, NI, EPI_STORE_F32, RH>(acc, e, wm * WM + lr, min(BM, M - tm * BM),
                                                  wcol + lc, BN, hs);
    return;
  }
  const int row0 = tm * BM + wm * WM + lr;
  if constexpr (KIND == EPI_STORE_F32) {
    Epi e = epi;
    e.out = (float*)epi.out + (int64_t)blockIdx.y * M * epi.ldo;
    plain_epilogue<SH, MI, NI, EK, RH>(acc, e, row0, M, tn * BN + wn * WN + lc, N);
  } else if constexpr (KIND == EPI_STORE || KIND == EPI_RESID) {
    if constexpr (kResPf) {
      if (rp.on) {
        __syncthreads();  // every wave's residual pieces have landed
        resid_lds_epilogue<SH, MI, NI, RH>(acc, epi, row0, M, tn * BN + wn * WN + lc, N, smem_raw,
                                       (K / kBK) & 1, wm * WM + lr, wn * WN + lc);
        return;
      }
    }
    plain_epilogue<SH, MI, NI, EK, RH>(acc, epi, row0, M, tn * BN + wn * WN + lc, N);
  } else if constexpr (KIND == EPI_SWIGLU) {
    swiglu_epilogue<SH, MI, NI, F32, RH>(acc, epi, row0, M, tn * (BN / 2) + wn * (WN / 2) + lc);
  } else {
    static_assert(PP, "the q/k/v epilogue pairs column groups as PingCols deals them");
    qkv_ping_epilogue<ML, KIND == EPI_QKV_NORM, F32>(acc, epi, smem_raw, wv, lane, tm * BM, tn * BN, M,
                                                 N);
  }
}

// LDS stages of a grouped tile form.
template <int BM, int BN, int WGM, int WGN, int SH>
constexpr int grouped_stages() {
  return is_ping<BM, BN, WGM, WGN, 2, SH>() && BM == 128 ? 3 : 2;
}

// Grouped expert GEMM.  Rows [seg[e], seg[e+1]) of the routed order belong to
// expert e; tile_off[e] .. tile_off[e+1]-1 are its M-tiles (BM rows each).  For
// the gate/up pass (EPI_SWIGLU) A row p is token perm[p] / top_k of A; for the
// down pass (EPI_STORE_F32) A row p is row p of A.  B of expert e starts at
// B + e * b_stride elements.  Output row = routed position p.
template <int BM, int BN, int WGM, int WGN, int EK, int SH = 32>
__global__ __launch_bounds__(WGM * WGN * 64) void gemm_grouped_kernel(
    const bf16* __restrict__ A, int lda, int a_rows, const int32_t* __restrict__ perm, int top_k,
    const bf16* __restrict__ B, int64_t b_stride, int N, int K,
    const int32_t* __restrict__ seg, const int32_t* __restrict__ tile_off, int n_experts,
    int tiles_n, Epi epi) {
  constexpr int S = grouped_stages<BM, BN, WGM, WGN, SH>();
  using ML = MainloopOf<BM, BN, WGM, WGN, S, SH>;
  constexpr bool PP = is_ping<BM, BN, WGM, WGN, S, SH>();
  constexpr int RH = ML::RH;
  using Geo = AccGeo<SH, ML::MI, ML::NI, RH>;
  constexpr int NW = ML::NW, MI = ML::MI, NI = ML::NI;
  constexpr int WM = PP ? 64 : BM / WGM, WN = BN / WGN;
  constexpr int KIND = EK & kEpiKindMask;
  constexpr bool F32 = (EK & kEpiF32) != 0;
  extern __shared__ __align__(16) char smem_raw[];
  GemmSmem<BM, BN, S>& sm = *reinterpret_cast<GemmSmem<BM, BN, S>*>(smem_raw);

  // The real tiles (tile_off[E] M-tiles x tiles_n) are dealt to the XCDs in
  // contiguous shares (block b runs on XCD b % 8), so an expert's M-tiles run
  // side by side on one XCD and share its weight k-slices in that L2;
  // surplus blocks exit.
  const int total = tile_off[n_experts] * tiles_n;
  const int xcd = blockIdx.x % kXcds, loc = blockIdx.x / kXcds;
  const int per = total / kXcds, rem = total % kXcds;
  if (loc >= per + (xcd < rem ? 1 : 0)) return;  // surplus block
  const int id = xcd * per + min(xcd, rem) + loc;
  const int tn = id % tiles_n, mt = id / tiles_n;
  int lo = 0, hi = n_experts;             // expert e with tile_off[e] <= mt < tile_off[e+1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (tile_off[mid] <= mt) lo = mid; else hi = mid;
  }
  const int e = lo;
  const int p0 = seg[e] + (mt - tile_off[e]) * BM;  // first routed row of this tile
  const int p_end = seg[e + 1];
  const int n_rows_b = KIND == EPI_SWIGLU ? 2 * epi.ffn : N;

  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / WGN, wn = wv % WGN;
  const __amdgpu_buffer_rsrc_t rsrc_a =
      __builtin_amdgcn_make_buffer_rsrc((void*)A, (short)0, (int)((int64_t)a_rows * lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(B + (int64_t)e * b_stride), (short)0, (int)((int64_t)n_rows_b * K * 2), 0x00020000);
  const int lrow = lane >> 3;
  uint32_t a_off[ML::A_BLK], b_off[ML::B_BLK];
#pragma unroll
  for (int j = 0; j < ML::A_BLK; ++j) {
    const int tr = (wv + NW * j) * 8 + lrow;
    const int p = p0 + tr;
    int src = -1;
    if (p < p_end) src = perm ? perm[p] / top_k : p;
    a_off[j] = (src >= 0 && src < a_rows)
                   ? (uint32_t)(((int64_t)src * lda + swz(tr, lane & 7) * 8) * 2)
                   : 0x80000000u;
  }
#pragma unroll
  for (int j = 0; j < ML::B_BLK; ++j) {
    const int tr = (wv + NW * j) * 8 + lrow;
    int gr;
    if constexpr (PP) gr = ML::b_row(KIND, tn, tr, epi.ffn, 0);
    else gr = b_row_of<BN, WN>(KIND, tn, tr, epi.ffn);
    b_off[j] = gr < n_rows_b ? (uint32_t)(((int64_t)gr * K + swz(tr, lane & 7) * 8) * 2) : 0x80000000u;
  }
  typename ML::acc_t acc[MI][NI];
  // Short-row tiles (decode) stream their weights at HBM rate with every
  // workgroup in flight at once; started at the same k-tile, all of them
  // would read at one offset modulo the weight row (4 KB rows for H = 2048),
  // so each rotates its k-loop by its own amount.  The prefill down
  // projection (fp32 output) gains from it too; the prefill gate/up, whose
  // tiles of one expert share their k-slices in L2, does not.
  const bool rotate = BM <= 32 || KIND == EPI_STORE_F32;
  const int kshift = rotate ? (int)(((unsigned)id * 7u) % (unsigned)(K / kBK)) : 0;
  ML::run_valid(p_end - p0, sm, rsrc_a, a_off, rsrc_b, b_off, K, wv, lane, acc, kshift);

  const int lr = Geo::lane_row(lane), lc = Geo::lane_col(lane);
  const int row0 = p0 + wm * WM + lr;
  if constexpr (KIND == EPI_SWIGLU)
    swiglu_epilogue<SH, MI, NI, F32, RH>(acc, epi, row0, p_end,
                                         tn * (BN / 2) + wn * (WN / 2) + lc);
  else
    plain_epilogue<SH, MI, NI, EK, RH>(acc, epi, row0, p_end, tn * BN + wn * WN + lc, N);
}

template <typename Kern>
static hipError_t opt_in_lds(Kern k, size_t smem, bool& done) {
  if (done) return hipSuccess;  // one-time opt-in to > 64 KB of LDS
  hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)smem);
  if (e == hipSuccess) done = true;
  return e;
}

// splits > 1 only with EPI_STORE_F32 (plane z of epi.out holds split z); K
// must then be a multiple of 64 * splits.
template <int BM, int BN, int WGM, int WGN, int EK, int S = 2, int SH = 32>
static hipError_t run_gemm(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                           const Epi& epi, hipStream_t s, int splits = 1) {
  const int tiles_m = cdiv(M, BM);
  const int tiles_n = (EK & kEpiKindMask) == EPI_SWIGLU ? cdiv(epi.ffn, BN / 2) : cdiv(N, BN);
  const size_t smem = sizeof(GemmSmem<BM, BN, S>);
  static bool attr_set = false;
  hipError_t e = opt_in_lds(gemm_kernel<BM, BN, WGM, WGN, EK, S, SH>, smem, attr_set);
  if (e != hipSuccess) return e;
  const int kc = K / splits;
  gemm_kernel<BM, BN, WGM, WGN, EK, S, SH><<<dim3(tiles_m * tiles_n, splits), WGM * WGN * 64, smem, s>>>(
      (const bf16*)A, lda, (const bf16*)B, ldb, M, N, K, kc, epi, tiles_m, tiles_n,
      tiles_m * tiles_n, 1, nullptr);
  return hipGetLastError();
}

int cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n = v;
    else
      n = 256;
  }
  return n;
}

// Bound for every large GEMM: the tail tiles times their splits never exceed
// one round (the CU count) of 256 x 256 fp32 tiles.
size_t gemm_tail_bytes() { return (size_t)cu_count() * 256 * 256 * sizeof(float); }

// Sum of a tail tile's split partials in split order + the epilogue.
// Workgroup (j, chunk): tail tile j (id full + j of the grouped order),
// elements [chunk * 2048, chunk * 2048 + 2048) of the tile (rotary pairs for
// q/k/v), 8 per thread.  Each thread loads its 8 elements' values of one
// split plane together, then every operand of the epilogue, before any
// store: tsplit + 1 memory round trips instead of one per element.
constexpr int kTailChunk = 2048;
constexpr int kTailPer = kTailChunk / 256;

// QKV: the q/k/v instantiation (its own kernel, so that the plain path's
// registers for every plane's values do not lower its occupancy).
template <int BM, int BN, bool F32, bool QKV>
__global__ __launch_bounds__(256) void tail_epi_kernel(const float* __restrict__ tail, int tsplit,
                                                       int full, int tiles_m, int tiles_n, int M,
                                                       int N, Epi epi) {
  using St = Store<F32>;
  using T = typename St::T;
  const int j = blockIdx.y;
  int tm, tn;
  tile_of_id(full + j, tiles_m, tiles_n, tm, tn);
  const float* __restrict__ tp = tail + (int64_t)j * tsplit * BM * BN;
  const int e0 = blockIdx.x * kTailChunk + threadIdx.x;
  // rows past M hold no partials: a workgroup of such rows has nothing to do,
  // and loads of a partly valid one stay within the valid rows
  constexpr int kRow = QKV ? BN / 2 : BN;  // elements per tile row
  if (tm * BM + (int)blockIdx.x * kTailChunk / kRow >= M) return;
  const int e_end = min(BM, M - tm * BM) * kRow;
  if constexpr (!QKV) {
    int idx[kTailPer];
    float v[kTailPer];
#pragma unroll
    for (int q = 0; q < kTailPer; ++q) {
      idx[q] = min(e0 + 256 * q, e_end - 1);
      v[q] = 0.f;
    }
    // every plane's values are loaded before the ordered sum (tsplit <=
    // kMaxTailSplit, a uniform bound), so the loads are in flight together
    float pv[kMaxTailSplit][kTailPer];
#pragma unroll
    for (int sp = 0; sp < kMaxTailSplit; ++sp)
#pragma unroll
      for (int q = 0; q < kTailPer; ++q)
        pv[sp][q] = sp < tsplit ? tp[(int64_t)sp * BM * BN + idx[q]] : 0.f;
#pragma unroll
    for (int sp = 0; sp < kMaxTailSplit; ++sp)
#pragma unroll
      for (int q = 0; q < kTailPer; ++q)
        if (sp < tsplit) v[q] += pv[sp][q];
    float res[kTailPer];
    if (epi.kind == EPI_RESID) {
#pragma unroll
      for (int q = 0; q < kTailPer; ++q) {
        const int row = min(tm * BM + idx[q] / BN, M - 1), col = min(tn * BN + idx[q] % BN, N - 1);
        res[q] = St::ld(epi.resid, (int64_t)row * epi.ldr + col);
      }
    }
#pragma unroll
    for (int q = 0; q < kTailPer; ++q) {
      const int e = e0 + 256 * q;
      const int row = tm * BM + e / BN, col = tn * BN + e % BN;
      if (e >= e_end || col >= N) continue;
      const float o = epi.kind == EPI_RESID ? v[q] + res[q] : v[q];
      St::st(epi.out, (int64_t)row * epi.ldo + col, o);
    }
    return;
  } else {
    // q/k/v + bias + RoPE + cache write: one thread per rotary pair (a head of
    // D columns lies inside one tile since BN is a multiple of D).
    const int Dh = epi.head_dim, half = Dh / 2;
    const int Hq = epi.n_q_heads, Hkv = epi.n_kv_heads;
    int rr[kTailPer], cc[kTailPer];
    float x1[kTailPer], x2[kTailPer];
#pragma unroll
    for (int q = 0; q < kTailPer; ++q) {
      const int e = min(e0 + 256 * q, e_end - 1);
      const int pc = e % (BN / 2);
      rr[q] = e / (BN / 2);
      cc[q] = (pc / half) * Dh + pc % half;  // first-half column in the tile
      x1[q] = x2[q] = 0.f;
    }
    // (plane by plane: loading every plane's pairs first needs twice the
    // registers of the plain path and was slower)
    for (int sp = 0; sp < tsplit; ++sp)
#pragma unroll
      for (int q = 0; q < kTailPer; ++q) {
        const float* pl = tp + (int64_t)sp * BM * BN + rr[q] * BN + cc[q];
        x1[q] += pl[0];
        x2[q] += pl[half];
      }
    float2 cs[kTailPer];
    int sl[kTailPer], tr[kTailPer];
    float b1[kTailPer], b2[kTailPer], g1[kTailPer], g2[kTailPer];
#pragma unroll
    for (int q = 0; q < kTailPer; ++q) {
      const int row = min(tm * BM + rr[q], M - 1), col = min(tn * BN + cc[q], N - 1);
      const int head = col / Dh, d = col % Dh;
      cs[q] = epi.rope[(int64_t)row * half + d];
      sl[q] = epi.tok_slot[row];
      tr[q] = epi.tok_row[row];
      b1[q] = epi.bias ? St::ld(epi.bias, col) : 0.f;
      b2[q] = epi.bias ? St::ld(epi.bias, col + half) : 0.f;
      const void* gp = head < Hq ? epi.q_norm : epi.k_norm;
      const bool n = epi.q_norm && head < Hq + Hkv;
      g1[q] = n ? St::ld(gp, d) : 1.f;
      g2[q] = n ? St::ld(gp, d + half) : 1.f;
    }
    // Per-head RMSNorm of q and k: a head's rotary pairs are `half` consecutive
    // elements, an aligned group of lanes, so its sum of squares is a group sum.
    float rs[kTailPer];
#pragma unroll
    for (int q = 0; q < kTailPer; ++q) {
      x1[q] += b1[q];
      x2[q] += b2[q];
      rs[q] = 1.f;
      if (epi.q_norm) {
        const float ss = group_sum(x1[q] * x1[q] + x2[q] * x2[q], half);
        rs[q] = 1.0f / sqrtf(ss / (float)Dh + epi.eps);
      }
    }
#pragma unroll
    for (int q = 0; q < kTailPer; ++q) {
      const int row = tm * BM + rr[q], col = tn * BN + cc[q];
      if (e0 + 256 * q >= e_end || col >= N) continue;
      const int head = col / Dh, d = col % Dh;
      float y1 = x1[q], y2 = x2[q];
      if (head < Hq + Hkv) {
        y1 *= rs[q] * g1[q];
        y2 *= rs[q] * g2[q];
        const float r1 = y1 * cs[q].x - y2 * cs[q].y;
        const float r2 = y2 * cs[q].x + y1 * cs[q].y;
        y1 = r1;
        y2 = r2;
      }
      T* dst;
      if (head < Hq) {
        dst = (T*)epi.q + ((int64_t)row * Hq + head) * Dh + d;
      } else {
        if (sl[q] < 0) continue;
        const int kvh = head < Hq + Hkv ? head - Hq : head - Hq - Hkv;
        T* cache = (T*)(head < Hq + Hkv ? epi.kc : epi.vc);
        dst = cache + (((int64_t)sl[q] * Hkv + kvh) * epi.max_seq + tr[q]) * Dh + d;
      }
      dst[0] = (T)y1;
      dst[half] = (T)y2;
    }
  }
}

// A GEMM whose last partial round of tiles (tail_tiles), one workgroup per CU, is
// cut in `t` K-parts (t > 1) or 128-row halves (t = 0) that fill it.
template <int BM, int BN, int WGM, int WGN, int EK, int S, int SH>
static hipError_t run_gemm_tail(const void* A, int lda, const void* B, int ldb, int M, int N,
                                int K, const Epi& epi, float* tail, hipStream_t s, int t) {
  constexpr int KIND = EK & kEpiKindMask;
  const int tiles_m = cdiv(M, BM);
  const int tiles_n = KIND == EPI_SWIGLU ? cdiv(epi.ffn, BN / 2) : cdiv(N, BN);
  const int total = tiles_m * tiles_n;
  if (t == 1) return run_gemm<BM, BN, WGM, WGN, EK, S, SH>(A, lda, B, ldb, M, N, K, epi, s);
  const int n_tail = tail_tiles(total, cu_count());
  const int full = total - n_tail;
  const size_t smem = sizeof(GemmSmem<BM, BN, S>);
  static bool attr_set = false;
  hipError_t e = opt_in_lds(gemm_kernel<BM, BN, WGM, WGN, EK, S, SH>, smem, attr_set);
  if (e != hipSuccess) return e;
  // t = 0: the tail tiles run as a second launch of their 128-row halves over
  // the whole K, with no fp32 partials and no reduction kernel.
  if constexpr (BM == 256) {
    if (t == 0) {
      if (full > 0) {
        gemm_kernel<BM, BN, WGM, WGN, EK, S, SH><<<full, WGM * WGN * 64, smem, s>>>(
            (const bf16*)A, lda, (const bf16*)B, ldb, M, N, K, K, epi, tiles_m, tiles_n, full, 1,
            nullptr);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
      const size_t hsmem = sizeof(GemmSmem<128, 256, 3>);
      static bool half_attr = false;
      e = opt_in_lds(gemm_kernel<128, 256, 2, 4, EK, 3, kTileSH>, hsmem, half_attr);
      if (e != hipSuccess) return e;
      gemm_kernel<128, 256, 2, 4, EK, 3, kTileSH><<<2 * n_tail, 512, hsmem, s>>>(
          (const bf16*)A, lda, (const bf16*)B, ldb, M, N, K, K, epi, tiles_m, tiles_n, full, 0,
          nullptr);
      return hipGetLastError();
    }
  }
  if (KIND == EPI_SWIGLU) return hipErrorInvalidValue;  // (its tail is never split in K)
  gemm_kernel<BM, BN, WGM, WGN, EK, S, SH><<<full + n_tail * t, WGM * WGN * 64, smem, s>>>(
      (const bf16*)A, lda, (const bf16*)B, ldb, M, N, K, K, epi, tiles_m, tiles_n, full, t, tail);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int elems = KIND == EPI_QKV || KIND == EPI_QKV_NORM ? BM * BN / 2 : BM * BN;
  constexpr bool kQkv = KIND == EPI_QKV || KIND == EPI_QKV_NORM;
  tail_epi_kernel<BM, BN, (EK & kEpiF32) != 0, kQkv>
      <<<dim3(cdiv(elems, kTailChunk), n_tail), 256, 0, s>>>(tail, t, full, tiles_m, tiles_n, M,
                                                             N, epi);
  return hipGetLastError();
}

template <int EK>
static hipError_t run_planned(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                              const Epi& epi, float* tail, hipStream_t s) {
  constexpr int KIND = EK & kEpiKindMask;
  const GemmPlan p = gemm_plan(M, KIND == EPI_SWIGLU ? 2 * epi.ffn : N, K, KIND == EPI_SWIGLU,
                               tail != nullptr, epi.routed != 0, cu_count());
  if (p.bm == 256)
    return run_gemm_tail<256, 256, 2, 4, EK, 2, kTileSH>(A, lda, B, ldb, M, N, K, epi, tail, s,
                                                            p.split);
  if (p.bn == 256)
    return run_gemm<128, 256, 2, 4, EK, 3, kTileSH>(A, lda, B, ldb, M, N, K, epi, s);
  return run_gemm_tail<128, 128, 2, 4, EK, 5, kTileSH>(A, lda, B, ldb, M, N, K, epi, tail, s, p.split);
}

hipError_t launch_gemm(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                       const Epi& epi, float* tail, hipStream_t s) {
  if (M == 0) return hipSuccess;
  if (epi.f32) {
    constexpr int F = kEpiF32;
    switch (epi.kind) {
      case EPI_RESID: return run_planned<EPI_RESID | F>(A, lda, B, ldb, M, N, K, epi, tail, s);
      case EPI_SWIGLU: return run_planned<EPI_SWIGLU | F>(A, lda, B, ldb, M, N, K, epi, tail, s);
      case EPI_QKV:
        if (epi.q_norm)
          return run_planned<EPI_QKV_NORM | F>(A, lda, B, ldb, M, N, K, epi, tail, s);
        return run_planned<EPI_QKV | F>(A, lda, B, ldb, M, N, K, epi, tail, s);
      default: return hipErrorInvalidValue;
    }
  }
  switch (epi.kind) {
    case EPI_STORE: return run_planned<EPI_STORE>(A, lda, B, ldb, M, N, K, epi, tail, s);
    case EPI_RESID: return run_planned<EPI_RESID>(A, lda, B, ldb, M, N, K, epi, tail, s);
    case EPI_SWIGLU: return run_planned<EPI_SWIGLU>(A, lda, B, ldb, M, N, K, epi, tail, s);
    case EPI_STORE_F32: return hipErrorInvalidValue;
    default:
      if (epi.q_norm) return run_planned<EPI_QKV_NORM>(A, lda, B, ldb, M, N, K, epi, tail, s);
      return run_planned<EPI_QKV>(A, lda, B, ldb, M, N, K, epi, tail, s);
  }
}

template <int BM, int BN, int WGM, int WGN, int EK, int SH = 32>
static hipError_t run_grouped(const void* A, int lda, int a_rows, const int32_t* perm, int top_k,
                              const void* B, int64_t b_stride, int N, int K, const int32_t* seg,
                              const int32_t* tile_off, int n_experts, int max_tiles_m,
                              const Epi& epi, hipStream_t s) {
  const int tiles_n = (EK & kEpiKindMask) == EPI_SWIGLU ? cdiv(epi.ffn, BN / 2) : cdiv(N, BN);
  const size_t smem = sizeof(GemmSmem<BM, BN, grouped_stages<BM, BN, WGM, WGN, SH>()>);
  static bool attr_set = false;
  hipError_t e = opt_in_lds(gemm_grouped_kernel<BM, BN, WGM, WGN, EK, SH>, smem, attr_set);
  if (e != hipSuccess) return e;
  gemm_grouped_kernel<BM, BN, WGM, WGN, EK, SH><<<max_tiles_m * tiles_n, WGM * WGN * 64, smem, s>>>(
      (const bf16*)A, lda, a_rows, perm, top_k, (const bf16*)B, b_stride, N, K, seg, tile_off,
      n_experts, tiles_n, epi);
  return hipGetLastError();
}

hipError_t launch_gemm_grouped(const void* A, int lda, int a_rows, const int32_t* perm, int top_k,
                               const void* B, int64_t b_stride, int N, int K, const int32_t* seg,
                               const int32_t* tile_off, int n_experts, int n_pairs,
                               int bm, const Epi& epi, hipStream_t s) {
  if (n_pairs == 0) return hipSuccess;
  if (bm != 32 && bm != 128 && bm != 256) return hipErrorInvalidValue;
  const int max_tiles_m = cdiv(n_pairs, bm) + n_experts;  // each expert adds <= 1 partial tile
  if (epi.f32 && epi.kind == EPI_SWIGLU) {
    constexpr int EK = EPI_SWIGLU | kEpiF32;
    if (bm == 32)
      return run_grouped<32, 256, 1, 4, EK>(A, lda, a_rows, perm, top_k, B, b_stride, N, K, seg,
                                            tile_off, n_experts, max_tiles_m, epi, s);
    if (bm == 256)
      return run_grouped<256, 256, 2, 4, EK, kTileSH>(A, lda, a_rows, perm, top_k, B, b_stride, N, K, seg,
                                             tile_off, n_experts, max_tiles_m, epi, s);
    return run_grouped<128, 256, 2, 4, EK, kTileSH>(A, lda, a_rows, perm, top_k, B, b_stride, N, K, seg,
                                           tile_off, n_experts, max_tiles_m, epi, s);
  }
  if (bm == 32) {
    if (epi.kind == EPI_SWIGLU)
      return run_grouped<32, 256, 1, 4, EPI_SWIGLU>(A, lda, a_rows, perm, top_k, B, b_stride, N, K,
                                                     seg, tile_off, n_experts, max_tiles_m, epi, s);
    return run_grouped<32, 256, 1, 4, EPI_STORE_F32>(A, lda, a_rows, perm, top_k, B, b_stride, N, K,
                                                      seg, tile_off, n_experts, max_tiles_m, epi, s);
  }
  if (bm == 256) {
    if (epi.kind == EPI_SWIGLU)
      return run_grouped<256, 256, 2, 4, EPI_SWIGLU, kTileSH>(A, lda, a_rows, perm, top_k, B, b_stride, N, K,
                                                      seg, tile_off, n_experts, max_tiles_m, epi, s);
    return run_grouped<256, 256, 2, 4, EPI_STORE_F32, kTileSH>(A, lda, a_rows, perm, top_k, B, b_stride, N,
                                                       K, seg, tile_off, n_experts, max_tiles_m, epi,
                                                       s);
  }
  if (epi.kind == EPI_SWIGLU)
    return run_grouped<128, 256, 2, 4, EPI_SWIGLU, kTileSH>(A, lda, a_rows, perm, top_k, B, b_stride, N, K,
                                                    seg, tile_off, n_experts, max_tiles_m, epi, s);
  return run_grouped<128, 256, 2, 4, EPI_STORE_F32, kTileSH>(A, lda, a_rows, perm, top_k, B, b_stride, N, K,
                                                     seg, tile_off, n_experts, max_tiles_m, epi, s);
}

// Split-K reduction: sum the fp32 partial planes [splits][M][N] in split
// order (deterministic) and apply the epilogue; one thread per output element
// (per intermediate column for SwiGLU, per rotary pair for q/k/v).
__global__ __launch_bounds__(256) void splitk_epi_kernel(const float* __restrict__ part,
                                                       int splits, int M, int N, Epi epi) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t MN = (int64_t)M * N;
  // All planes' values are loaded before the ordered sum (splits <= 16), so
  // the loads are in flight together.
  auto sum = [&](int row, int col) {
    const float* q = part + (int64_t)row * N + col;
    float t[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) t[s] = s < splits ? q[s * MN] : 0.f;
    float v = 0.f;
#pragma unroll
    for (int s = 0; s < 16; ++s) v += t[s];
    return v;
  };
  if (epi.kind == EPI_STORE || epi.kind == EPI_RESID) {
    if (gid >= MN) return;
    const int row = (int)(gid / N), col = (int)(gid % N);
    float v = sum(row, col);
    if (epi.kind == EPI_RESID) v += bf2f(((const bf16*)epi.resid)[(int64_t)row * epi.ldr + col]);
    ((bf16*)epi.out)[(int64_t)row * epi.ldo + col] = f2bf(v);
  } else if (epi.kind == EPI_SWIGLU) {
    const int F = epi.ffn;
    if (gid >= (int64_t)M * F) return;
    const int row = (int)(gid / F), f = (int)(gid % F);
    const float g = sum(row, f), u = sum(row, F + f);
    ((bf16*)epi.out)[(int64_t)row * epi.ldo + f] = f2bf(silu(g) * u);
  } else {  // EPI_QKV: one thread per rotary pair
    const int D = epi.head_dim, half = D / 2;
    const int Hq = epi.n_q_heads, Hkv = epi.n_kv_heads;
    const int pairs = (Hq + 2 * Hkv) * half;
    // lanes past the end compute on a clamped pair (their group is whole:
    // M pairs is a multiple of half) and store nothing
    const bool live = gid < (int64_t)M * pairs;
    const int64_t g = live ? gid : (int64_t)M * pairs - 1;
    const int row = (int)(g / pairs), p = (int)(g % pairs);
    const int head = p / half, d = p % half;
    const int col = head * D + d;
    float x1 = sum(row, col), x2 = sum(row, col + half);
    if (epi.bias) {
      x1 += bf2f(((const bf16*)epi.bias)[col]);
      x2 += bf2f(((const bf16*)epi.bias)[col + half]);
    }
    if (epi.q_norm) {
      // per-head RMSNorm of q and k: a head's pairs are an aligned group of
      // `half` lanes (D / 2 = 32 or 64)
      const float ss = group_sum(x1 * x1 + x2 * x2, half);
      if (head < Hq + Hkv) {
        const bf16* gp = (const bf16*)(head < Hq ? epi.q_norm : epi.k_norm);
        const float r = 1.0f / sqrtf(ss / (float)D + epi.eps);
        x1 *= r * bf2f(gp[d]);
        x2 *= r * bf2f(gp[d + half]);
      }
    }
    if (!live) return;
    if (head < Hq + Hkv) {
      const float2 cs = epi.rope[(int64_t)row * half + d];
      const float y1 = x1 * cs.x - x2 * cs.y;
      const float y2 = x2 * cs.x + x1 * cs.y;
      x1 = y1;
      x2 = y2;
    }
    if (head < Hq) {
      bf16* qp = (bf16*)epi.q + ((int64_t)row * Hq + head) * D + d;
      qp[0] = f2bf(x1);
      qp[half] = f2bf(x2);
    } else {
      const int sl = epi.tok_slot[row];
      if (sl < 0) return;
      const int kvh = head < Hq + Hkv ? head - Hq : head - Hq - Hkv;
      bf16* cache = (bf16*)(head < Hq + Hkv ? epi.kc : epi.vc);
      bf16* cp = cache + (((int64_t)sl * Hkv + kvh) * epi.max_seq + epi.tok_row[row]) * D + d;
      cp[0] = f2bf(x1);
      cp[half] = f2bf(x2);
    }
  }
}

// Split-K reduction fused with the residual add and the RMSNorm that follows
// it (the O projection of a short batch): one workgroup per row sums the
// planes in split order and adds the residual (x1, stored in bf16), then
// normalises the stored row into y = x1 / sqrt(mean(x1^2) + eps) * g.
constexpr int kNormRowThreads = 256;
constexpr int kNormRowChunks = 8;  // 4-float chunks per thread: N <= 256 * 4 * 8

__global__ __launch_bounds__(kNormRowThreads) void splitk_resid_norm_kernel(
    const float* __restrict__ part, int splits, int M, int N, const bf16* __restrict__ resid,
    int ldr, bf16* __restrict__ out, int ldo, const bf16* __restrict__ g, bf16* __restrict__ y,
    float eps) {
  const int row = blockIdx.x, tid = threadIdx.x;
  const int64_t MN = (int64_t)M * N;
  const int nch = N / 4;
  f32x4 v[kNormRowChunks];
  float res[kNormRowChunks][4], gg[kNormRowChunks][4];
  // Every operand of the row first (chunk indices clamped: no branch around
  // the loads), then the ordered plane sums.
#pragma unroll
  for (int c = 0; c < kNormRowChunks; ++c) {
    const int ch = min(tid + c * kNormRowThreads, nch - 1);
    const bf16* rp = resid + (int64_t)row * ldr + ch * 4;
    const bf16* gp = g + ch * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      res[c][e] = bf2f(rp[e]);
      gg[c][e] = bf2f(gp[e]);
    }
    v[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // planes in groups of four: a group's loads are in flight together, then
  // added in plane order
  for (int sp0 = 0; sp0 < splits; sp0 += 4) {
    f32x4 t[4][kNormRowChunks];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < kNormRowChunks; ++c) {
        const int ch = min(tid + c * kNormRowThreads, nch - 1);
        const int sp = min(sp0 + j, splits - 1);  // past the last plane: re-read, dropped
        t[j][c] = *(const f32x4*)(part + sp * MN + (int64_t)row * N + ch * 4);
      }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < kNormRowChunks; ++c)
        if (sp0 + j < splits) v[c] += t[j][c];
  }
  float ss = 0.f;
  bf16 x1[kNormRowChunks][4];
#pragma unroll
  for (int c = 0; c < kNormRowChunks; ++c) {
    const bool ok = tid + c * kNormRowThreads < nch;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x1[c][e] = f2bf(v[c][e] + res[c][e]);
      const float f = bf2f(x1[c][e]);
      if (ok) ss += f * f;
    }
  }
  __shared__ float red[kNormRowThreads / 64];
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int w = 0; w < kNormRowThreads / 64; ++w) ss += red[w];
  const float r = 1.0f / sqrtf(ss / (float)N + eps);
#pragma unroll
  for (int c = 0; c < kNormRowChunks; ++c) {
    const int ch = tid + c * kNormRowThreads;
    if (ch >= nch) continue;
    bf16x4 o, h;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = x1[c][e];
      h[e] = f2bf(bf2f(x1[c][e]) * r * gg[c][e]);
    }
    *(bf16x4*)(out + (int64_t)row * ldo + ch * 4) = o;
    *(bf16x4*)(y + (int64_t)row * N + ch * 4) = h;
  }
}

// Decode projections of up to 128 rows that do not run as weight streams
// (stream_rows).  The arithmetic intensity is ~M flop
// per weight byte, so the weight stream from HBM sets the time: skinny
// 64 x 64 tiles (two or four waves) give ~600 workgroups on the large
// projections -- every one resident at once, each a short run of weight rows,
// which keeps the HBM pages streaming -- and split-K multiplies the
// workgroups of the narrow projections until ~200 are in flight.  Without a
// split the epilogue is fused; with one, fp32 partial planes go to the
// workspace and splitk_epi_kernel finishes.
// q/k/v always splits (its fused epilogue needs a whole head per wave).  The
// split runs of up to two workgroups per CU keep four k-tiles in LDS (three
// in flight), the rest two.  For q/k/v at 64 rows, 4 splits with four stages
// beat 8 with two: its partial planes are halved, and so is what they leave
// dirty in the caches just before the attention streams the KV cache.  Over
// 128-row tiles every split run likewise takes half the workgroups (~100)
// with three stages (two workgroups per CU): fewer partial planes ahead of
// the attention and of the weight streams that follow.
constexpr int kSkinnyBN = 64;

static int skinny_bm(int M) { return M <= 64 ? 64 : 128; }

static int skinny_splits(int M, int N, int K, int kind) {
  const int tiles = cdiv(M, skinny_bm(M)) * cdiv(N, kSkinnyBN);
  const int target = M > 64 ? 100 : 200;
  int s = 1;
  while ((tiles * s < target || (kind == EPI_QKV && s == 1)) && s < 16 &&
         K % (kBK * 2 * s) == 0)
    s *= 2;
  return s;
}

// fp32 partial planes [splits][M][N] of a short batch.
static hipError_t run_skinny_planes(const void* A, int lda, const void* B, int ldb, int M, int N,
                                    int K, float* part, int splits, int kind, hipStream_t s) {
  Epi pe{};
  pe.kind = EPI_STORE_F32;
  pe.out = part;
  pe.ldo = N;
  if (M > 64) {
    if (cdiv(N, kSkinnyBN) * splits <= 2 * cu_count())
      return run_gemm<128, kSkinnyBN, 4, 1, EPI_STORE_F32, 3>(A, lda, B, ldb, M, N, K, pe, s, splits);
    return run_gemm<128, kSkinnyBN, 4, 1, EPI_STORE_F32>(A, lda, B, ldb, M, N, K, pe, s, splits);
  }
  if (cdiv(N, kSkinnyBN) * splits <= 2 * cu_count())
    return run_gemm<64, kSkinnyBN, 2, 1, EPI_STORE_F32, 4>(A, lda, B, ldb, M, N, K, pe, s, splits);
  return run_gemm<64, kSkinnyBN, 2, 1, EPI_STORE_F32>(A, lda, B, ldb, M, N, K, pe, s, splits);
}

static bool streams(int M, int N, int K, int kind) {
  return M <= stream_rows(N, K, kind == EPI_SWIGLU || kind == EPI_QKV);
}

// fp32 planes [planes][M][N] that a short projection leaves in `part` for a
// second kernel, 0 if its own epilogue finishes it.  norm: that kernel also
// normalises (the q/k norm, RMSNorm after a residual), which needs whole heads
// or rows; a stream needs a plane for nothing else.
static int skinny_planes(int M, int N, int K, int kind, bool norm) {
  if (streams(M, N, K, kind)) return norm ? 1 : 0;
  const int s = skinny_splits(M, N, K, kind);
  return s > 1 ? s : 0;
}

size_t skinny_partial_bytes(int M, int N, int K, int kind, bool norm) {
  return (size_t)skinny_planes(M, N, K, kind, norm) * M * N * sizeof(float);
}

template <int BM, int WGM>
static hipError_t run_skinny(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                             const Epi& epi, float* part, int splits, hipStream_t s) {
  if (splits == 1) {
    switch (epi.kind) {
      case EPI_STORE: return run_gemm<BM, kSkinnyBN, WGM, 1, EPI_STORE>(A, lda, B, ldb, M, N, K, epi, s);
      case EPI_RESID: return run_gemm<BM, kSkinnyBN, WGM, 1, EPI_RESID>(A, lda, B, ldb, M, N, K, epi, s);
      case EPI_SWIGLU: return run_gemm<BM, kSkinnyBN, WGM, 1, EPI_SWIGLU>(A, lda, B, ldb, M, N, K, epi, s);
      case EPI_STORE_F32:
        return run_gemm<BM, kSkinnyBN, WGM, 1, EPI_STORE_F32>(A, lda, B, ldb, M, N, K, epi, s);
      default: return hipErrorInvalidValue;
    }
  }
  hipError_t e = run_skinny_planes(A, lda, B, ldb, M, N, K, part, splits, epi.kind, s);
  if (e != hipSuccess) return e;
  int64_t n_out;
  if (epi.kind == EPI_SWIGLU) n_out = (int64_t)M * epi.ffn;
  else if (epi.kind == EPI_QKV) n_out = (int64_t)M * (epi.n_q_heads + 2 * epi.n_kv_heads) * (epi.head_dim / 2);
  else n_out = (int64_t)M * N;
  splitk_epi_kernel<<<(unsigned)((n_out + 255) / 256), 256, 0, s>>>(part, splits, M, N, epi);
  return hipGetLastError();
}

static hipError_t run_stream_plane(const void* A, int lda, const void* B, int ldb, int M, int N,
                                   int K, float* plane, hipStream_t s) {
  Epi pe{};
  pe.kind = EPI_STORE_F32;
  pe.out = plane;
  pe.ldo = N;
  return launch_stream(A, lda, B, ldb, M, N, K, pe, s);
}

hipError_t launch_skinny(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                         const Epi& epi, float* part, hipStream_t s) {
  if (M == 0) return hipSuccess;
  const int planes = skinny_planes(M, N, K, epi.kind, epi.kind == EPI_QKV && epi.q_norm);
  if (streams(M, N, K, epi.kind)) {
    if (planes == 0) return launch_stream(A, lda, B, ldb, M, N, K, epi, s);
    hipError_t e = run_stream_plane(A, lda, B, ldb, M, N, K, part, s);
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)M * (epi.n_q_heads + 2 * epi.n_kv_heads) * (epi.head_dim / 2);
    splitk_epi_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(part, 1, M, N, epi);
    return hipGetLastError();
  }
  if (planes == 0 && epi.kind == EPI_QKV)
    return launch_gemm(A, lda, B, ldb, M, N, K, epi, nullptr, s);
  const int splits = planes > 0 ? planes : 1;
  if (M <= 64) return run_skinny<64, 2>(A, lda, B, ldb, M, N, K, epi, part, splits, s);
  return run_skinny<128, 4>(A, lda, B, ldb, M, N, K, epi, part, splits, s);
}

bool skinny_resid_norm_fused(int M, int N, int K) {
  return M <= 128 && M > 0 && N % 4 == 0 && N <= kNormRowThreads * 4 * kNormRowChunks &&
         skinny_planes(M, N, K, EPI_RESID, true) > 0;
}

hipError_t launch_skinny_resid_norm(const void* A, int lda, const void* B, int ldb, int M, int N,
                                    int K, const void* resid, int ldr, void* out, int ldo,
                                    const void* g, void* y, float eps, float* part, hipStream_t s) {
  if (M == 0) return hipSuccess;
  const int planes = skinny_planes(M, N, K, EPI_RESID, true);
  const hipError_t e = streams(M, N, K, EPI_RESID)
                           ? run_stream_plane(A, lda, B, ldb, M, N, K, part, s)
                           : run_skinny_planes(A, lda, B, ldb, M, N, K, part, planes, EPI_RESID, s);
  if (e != hipSuccess) return e;
  splitk_resid_norm_kernel<<<M, kNormRowThreads, 0, s>>>(part, planes, M, N, (const bf16*)resid,
                                                        ldr, (bf16*)out, ldo, (const bf16*)g,
                                                        (bf16*)y, eps);
  return hipGetLastError();
}

int gemm_planes_splits(int M, int N, int K) {
  const int tiles = cdiv(M, 64) * cdiv(N, kSkinnyBN);
  int s = 1;
  while (tiles * s < 400 && s < 16 && K % (kBK * 2 * s) == 0) s *= 2;
  return s;
}

hipError_t launch_gemm_planes(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                              float* planes, int splits, hipStream_t s) {
  if (M == 0) return hipSuccess;
  Epi pe{};
  pe.kind = EPI_STORE_F32;
  pe.out = planes;
  pe.ldo = plane_ld(N);
  return run_gemm<64, kSkinnyBN, 2, 1, EPI_STORE_F32>(A, lda, B, ldb, M, N, K, pe, s, splits);
}

}  // namespace tri
