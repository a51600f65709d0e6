// Short-batch projections (at most 16 tokens) as weight streams: C[M,N] = A[M,K]
// B[N,K]^T with the layer's epilogues, bf16 operands, fp32 accumulation.
//
// Such a product does M flops per weight byte, so it takes the time of reading
// the weights once.  What a stream needs is bytes in flight on every CU from
// the first microsecond to the last, and waves that do not wait for each
// other:
//  * a workgroup takes blocks of 16 RB weight rows over the whole K; its W waves
//    take the k-tiles (64 k, one 128-byte line of every row) in turn, so the
//    workgroup reads W neighbouring lines of each row at a time;
//  * each wave keeps D k-tiles in flight in an LDS ring of its own (direct
//    loads, 16-byte chunks swizzled as in the GEMM tiles: weights, and the
//    tokens' lines, L2 hits), ordered by its own vmcnt: the only barriers are
//    the two around a block's sum, and the next block's tiles load under them;
//  * the waves' partial sums meet in LDS, in wave order, and the epilogue is
//    fused: no partial planes in memory and no reduction kernel.
// Weight rows are the MFMA's row operand (16 x 16 x 32), tokens its columns.
//
// Bound by HBM: a pure stream of the same matrices takes 43 us (gate/up of the 7B
// layer, 271 MB), 23 us (down), 7 us (q/k/v); one token's step, same box: gate/up
// 52.3 + 3.9 (norm) -> 46 us with its norm, q/k/v 15.6 -> 9.6, down 30.8 -> 25, O 11.5
// + norm -> 8 us, the step 131 -> 110 us; the Talker's step 50 -> 34 us.
// Beyond 16 tokens the activations become a stream as large as the weights'
// (23 tokens: down 32 -> 38 us, 64 tokens: gate/up 62 -> 78 us), and the
// workgroup-wide 64-row tiles of the skinny GEMM are faster; so they are, with
// fewer tokens, for a narrow matrix with a long K (stream_rows).
#include "common.hpp"
#include "kernels.hpp"

namespace tri {

constexpr int kSBK = 64;  // k per k-tile

// Workgroup `blk`'s local row r (0 .. 16 RB - 1) -> weight row.  SwiGLU: 16 gate
// rows, then the matching up rows; q/k/v: 16 rows of a head's first half, then
// their rotary partners.
template <int KIND, int RB>
__device__ __forceinline__ int stream_row(int blk, int r, const Epi& epi) {
  if constexpr (KIND == EPI_SWIGLU) {
    const int f = blk * 16 + (r & 15);
    return r < 16 ? f : epi.ffn + f;
  } else if constexpr (KIND == EPI_QKV) {
    const int per = epi.head_dim / 32;  // workgroups per head
    return (blk / per) * epi.head_dim + (blk % per) * 16 + (r & 15) +
           (r < 16 ? 0 : epi.head_dim / 2);
  } else {
    return blk * 16 * RB + r;
  }
}

// One output group of a thread: four columns of a token row (and, for paired
// kinds, the four partner columns).  Its operands are loaded at the start of
// the block, under the weight stream.
template <int KIND>
struct StreamOut {
  f32x4 cs[2];            // (cos, sin) of the four rotary pairs
  bf16x4 b1, b2;          // bias, or the residual in b1
  int slot, crow;         // cache panel and row of the token
  int head, d;

  __device__ __forceinline__ void load(const Epi& epi, int blk, int row, int col) {
    if constexpr (KIND == EPI_QKV) {
      const int Dh = epi.head_dim, half = Dh / 2, per = Dh / 32;
      head = blk / per;
      d = (blk % per) * 16 + col;
      const float2* rp = epi.rope + (int64_t)row * half + d;
      cs[0] = *(const f32x4*)rp;
      cs[1] = *(const f32x4*)(rp + 2);
      slot = epi.tok_slot[row];
      crow = epi.tok_row[row];
      b1 = b2 = bf16x4{};
      if (epi.bias) {
        const bf16* bp = (const bf16*)epi.bias + head * Dh + d;
        b1 = *(const bf16x4*)bp;
        b2 = *(const bf16x4*)(bp + half);
      }
    } else if constexpr (KIND == EPI_RESID) {
      b1 = *(const bf16x4*)((const bf16*)epi.resid + (int64_t)row * epi.ldr + col);
    }
  }
  // x1: the group's sums, x2: its partner's (paired kinds)
  __device__ __forceinline__ void store(const Epi& epi, int row, int col, f32x4 x1, f32x4 x2) {
    if constexpr (KIND == EPI_SWIGLU) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = f2bf(silu(x1[e]) * x2[e]);
      *(bf16x4*)((bf16*)epi.out + (int64_t)row * epi.ldo + col) = o;
    } else if constexpr (KIND == EPI_QKV) {
      const int Dh = epi.head_dim, half = Dh / 2, Hq = epi.n_q_heads, Hkv = epi.n_kv_heads;
      bf16x4 o1, o2;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float y1 = x1[e] + bf2f(b1[e]), y2 = x2[e] + bf2f(b2[e]);
        if (head < Hq + Hkv) {
          const float c = cs[e >> 1][2 * (e & 1)], sn = cs[e >> 1][2 * (e & 1) + 1];
          const float z1 = y1 * c - y2 * sn;
          y2 = y2 * c + y1 * sn;
          y1 = z1;
        }
        o1[e] = f2bf(y1);
        o2[e] = f2bf(y2);
      }
      bf16* p = (bf16*)epi.q + ((int64_t)row * Hq + head) * Dh + d;
      if (head >= Hq) {
        if (slot < 0) return;
        const int kvh = head < Hq + Hkv ? head - Hq : head - Hq - Hkv;
        p = (bf16*)(head < Hq + Hkv ? epi.kc : epi.vc) +
            (((int64_t)slot * Hkv + kvh) * epi.max_seq + crow) * Dh + d;
      }
      *(bf16x4*)p = o1;
      *(bf16x4*)(p + half) = o2;
    } else if constexpr (KIND == EPI_STORE_F32) {
      *(f32x4*)((float*)epi.out + (int64_t)row * epi.ldo + col) = x1;
    } else {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        o[e] = f2bf(KIND == EPI_RESID ? x1[e] + bf2f(b1[e]) : x1[e]);
      *(bf16x4*)((bf16*)epi.out + (int64_t)row * epi.ldo + col) = o;
    }
  }
};

// Workgroup b takes the blocks of 16 RB weight rows b, b + grid, ...: one
// continuous stream per wave, the next block's first tiles loading while the
// current one's last are multiplied and summed.
//
// NORM: A is not read as it is but RMS-normalised (gains g) by every workgroup
// for itself, while its first weight tiles are on their way, into an LDS panel
// [M][K] (chunks at chunk ^ (row % 8) within a k-tile); workgroup 0 also writes
// the normalised rows to `h`.  For the few rows of a single user's step that
// is less work than one more kernel.
template <int AR, int RB, int W, int D, int KIND, bool NORM>
__global__ __launch_bounds__(W * 64) void stream_gemm_kernel(const bf16* __restrict__ A, int lda,
                                                            const bf16* __restrict__ B, int ldb,
                                                            int M, int N, int n_rows_b, int K,
                                                            int n_blk, Epi epi, StreamNorm nrm) {
  constexpr int LW = 2 * RB, LA = NORM ? 0 : AR / 8, LT = LW + LA;  // loads per k-tile
  constexpr int WT = 16 * RB * kSBK, TILE = WT + LA * 8 * kSBK;     // elements of a k-tile
  static_assert((D - 1) * LT < 64, "vmcnt counts up to 63");
  constexpr bool PAIR = KIND == EPI_SWIGLU || KIND == EPI_QKV;  // row block 0 pairs with 1
  constexpr int NB = PAIR ? 1 : RB;                             // output groups of 16 columns
  static_assert((PAIR ? RB == 2 : true) && NB * 64 <= W * 64, "one output group per thread");
  extern __shared__ __align__(16) char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lg = lane >> 4;
  bf16* const ring = (bf16*)smem_raw + wv * D * TILE;
  float* const red = (float*)(smem_raw + W * D * TILE * 2);  // [W][RB][16 tokens][16 columns]
  bf16* const panel = (bf16*)(red + W * RB * 256);

  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      (void*)A, (short)0, (int)((int64_t)M * lda * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(
      (void*)B, (short)0, (int)((int64_t)n_rows_b * ldb * 2), 0x00020000);
  uint32_t w_off[LW], a_off[LA > 0 ? LA : 1];
  auto block_rows = [&](int blk) {
#pragma unroll
    for (int j = 0; j < LW; ++j) {
      const int r = 8 * j + (lane >> 3), g = stream_row<KIND, RB>(blk, r, epi);
      w_off[j] = blk < n_blk && g < n_rows_b
                     ? (uint32_t)(((int64_t)g * ldb + swz(r, lane & 7) * 8) * 2)
                     : 0x80000000u;
    }
  };
#pragma unroll
  for (int j = 0; j < LA; ++j) {
    const int r = 8 * j + (lane >> 3);
    a_off[j] = r < M ? (uint32_t)(((int64_t)r * lda + swz(r, lane & 7) * 8) * 2) : 0x80000000u;
  }
  // The wave's i-th k-tile of a block is wv + W i.  The stream runs D tiles
  // ahead; past the last block, and in a wave with no k-tile at all (fewer
  // k-tiles than waves), its loads are out of range (zeros, no traffic), which
  // keeps the load count uniform.
  const int KT = K / kSBK;
  const int nt = wv < KT ? (KT - wv + W - 1) / W : 0;
  int ib = blockIdx.x, ii = 0, islot = 0;  // the next tile to load
  auto issue = [&]() {
    const uint32_t kill = ib < n_blk && nt > 0 ? 0u : 0x80000000u;
    const int kb = (wv + W * ii) * kSBK * 2;
    bf16* dst = ring + islot * TILE;
#pragma unroll
    for (int j = 0; j < LW; ++j) buffer_load_lds16(rb, dst + j * 512, w_off[j] | kill, kb);
#pragma unroll
    for (int j = 0; j < LA; ++j) buffer_load_lds16(ra, dst + WT + j * 512, a_off[j] | kill, kb);
    islot = islot + 1 == D ? 0 : islot + 1;
    if (++ii >= nt) {
      ii = 0;
      ib += gridDim.x;
      block_rows(ib);
    }
  };
  // Fragment of k-step ks: row lr, chunk 4 ks + lg (of eight token rows, the
  // columns past them repeat the first ones and are not written).
  const int ar = NORM ? min(lr, M - 1) : AR < 16 ? lr & 7 : lr;
  uint32_t f_off[2], t_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    f_off[ks] = (uint32_t)((lr * kSBK + swz(lr, 4 * ks + lg) * 8) * 2);
    t_off[ks] = NORM ? (uint32_t)((ar * K + ((4 * ks + lg) ^ (ar & 7)) * 8) * 2)
                     : (uint32_t)((WT + ar * kSBK + swz(ar, 4 * ks + lg) * 8) * 2);
  }
  block_rows(ib);
  if constexpr (NORM) {
    // x and g are requested ahead of the weights (loads return in order); a wave
    // per row, as in the RMSNorm kernel
    constexpr int XC = kStreamNormMaxCols / 512;  // 16-byte chunks per lane
    const int nch = K / 8;
    Pack8 xv[XC], gv[XC];
    auto load_row = [&](int m) {
#pragma unroll
      for (int c = 0; c < XC; ++c) {
        const int ch = min(lane + 64 * c, nch - 1);
        xv[c].u = ldg16(A + (int64_t)m * lda + ch * 8);
        gv[c].u = ldg16(nrm.g + ch * 8);
      }
    };
    load_row(min(wv, M - 1));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < D; ++d) issue();
    __builtin_amdgcn_sched_barrier(0);
    for (int m = wv; m < M; m += W) {
      if (m != wv) load_row(m);
      float ss = 0.f;
#pragma unroll
      for (int c = 0; c < XC; ++c)
        if (lane + 64 * c < nch)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float f = bf2f(xv[c].e[e]);
            ss += f * f;
          }
      ss = wave_sum(ss);
      const float r = 1.0f / sqrtf(ss / (float)K + nrm.eps);
#pragma unroll
      for (int c = 0; c < XC; ++c) {
        const int ch = lane + 64 * c;
        if (ch < nch) {
          Pack8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o.e[e] = f2bf(bf2f(xv[c].e[e]) * r * bf2f(gv[c].e[e]));
          *(u32x4*)(panel + m * K + (ch ^ (m & 7)) * 8) = o.u;
          if (blockIdx.x == 0) stg16(nrm.h + (int64_t)m * K + ch * 8, o.u);
        }
      }
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d) issue();
  }
  // this thread's output group: row orow, columns 4 (tid % 4) of group ob
  const int ob = threadIdx.x >> 6, orow = (threadIdx.x >> 2) & 15, oc = 4 * (threadIdx.x & 3);
  int slot = 0;
  for (int blk = blockIdx.x; blk < n_blk; blk += gridDim.x) {
    const int ocol = PAIR ? (KIND == EPI_SWIGLU ? blk * 16 + oc : oc) : blk * 16 * RB + 16 * ob + oc;
    // (N and ffn are multiples of 4)
    const bool out_ok = ob < NB && orow < M &&
                        (KIND == EPI_QKV || ocol < (KIND == EPI_SWIGLU ? epi.ffn : N));
    StreamOut<KIND> so;
    if (out_ok) so.load(epi, blk, orow, ocol);
    f32x4 acc[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) acc[b] = f32x4{0.f};
    for (int i = 0; i < nt; ++i) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * LT) : "memory");  // tile i landed
      bf16x8 wf[RB][2], av[2];
      const char* p = (const char*)(ring + slot * TILE);
      const char* q = NORM ? (const char*)panel + (wv + W * i) * kSBK * 2 : p;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        av[ks] = *(const bf16x8*)(q + t_off[ks]);
#pragma unroll
        for (int b = 0; b < RB; ++b)
          wf[b][ks] = *(const bf16x8*)(p + f_off[ks] + b * 16 * kSBK * 2);
      }
      // the slot's fragments are in registers: it may be filled again
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue();
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int b = 0; b < RB; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[b][ks], av[ks], acc[b], 0, 0, 0);
      slot = slot + 1 == D ? 0 : slot + 1;
    }
    // the waves' partial sums, added in wave order
#pragma unroll
    for (int b = 0; b < RB; ++b) *(f32x4*)&red[((wv * RB + b) * 16 + lr) * 16 + 4 * lg] = acc[b];
    __syncthreads();
    if (out_ok) {
      auto sum = [&](int b) {
        const float* p = &red[(b * 16 + orow) * 16 + oc];
        f32x4 v = *(const f32x4*)p;
#pragma unroll
        for (int w = 1; w < W; ++w) v += *(const f32x4*)(p + w * RB * 256);
        return v;
      };
      so.store(epi, orow, ocol, sum(PAIR ? 0 : ob), PAIR ? sum(RB - 1) : f32x4{});
    }
    __syncthreads();  // the sums are read before the next block's are written
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may land after the end
}

template <int AR, int RB, int W, int D, int KIND, bool NORM = false>
static hipError_t run_stream(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                             const Epi& epi, hipStream_t s, const StreamNorm& nrm = StreamNorm{}) {
  const int n_rows_b = KIND == EPI_SWIGLU ? 2 * epi.ffn : N;
  const int n_blk = cdiv(n_rows_b, 16 * RB);
  constexpr size_t fixed = (size_t)W * D * (16 * RB + (NORM ? 0 : AR)) * kSBK * 2 +
                           (size_t)W * RB * 1024;
  constexpr size_t most = fixed + (NORM ? kStreamNormMaxElems * 2 : 0);
  static_assert(most <= 160 * 1024, "LDS of a CU");
  const size_t smem = fixed + (NORM ? (size_t)M * K * 2 : 0);
  static bool done = false;
  if (!done) {
    hipError_t e = hipFuncSetAttribute((const void*)stream_gemm_kernel<AR, RB, W, D, KIND, NORM>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
    if (e != hipSuccess) return e;
    done = true;
  }
  // as many workgroups as are resident at once (LDS), each streaming its blocks
  const int resident = cu_count() * (int)((160 * 1024) / smem);
  const int grid = n_blk < resident ? n_blk : resident;
  stream_gemm_kernel<AR, RB, W, D, KIND, NORM><<<grid, W * 64, smem, s>>>(
      (const bf16*)A, lda, (const bf16*)B, ldb, M, N, n_rows_b, K, n_blk, epi, nrm);
  return hipGetLastError();
}

// Forms.  Two row blocks of 16 per workgroup block where the epilogue pairs rows
// or one would need several rounds of workgroups, one otherwise; four waves
// where there are blocks for two workgroups per CU, else eight.
template <int AR>
static hipError_t stream_rows(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                              const Epi& epi, hipStream_t s) {
  constexpr int D2 = 3, D1 = AR == 8 ? 6 : 4;  // k-tiles in flight for RB = 2, 1
  switch (epi.kind) {
    case EPI_SWIGLU: return run_stream<AR, 2, 4, D2, EPI_SWIGLU>(A, lda, B, ldb, M, N, K, epi, s);
    case EPI_QKV: return run_stream<AR, 2, 8, D2, EPI_QKV>(A, lda, B, ldb, M, N, K, epi, s);
    case EPI_RESID: return run_stream<AR, 1, 8, D1, EPI_RESID>(A, lda, B, ldb, M, N, K, epi, s);
    case EPI_STORE_F32:
      if (N > 16 * cu_count())
        return run_stream<AR, 2, 8, D2, EPI_STORE_F32>(A, lda, B, ldb, M, N, K, epi, s);
      return run_stream<AR, 1, 8, D1, EPI_STORE_F32>(A, lda, B, ldb, M, N, K, epi, s);
    case EPI_STORE:
      if (N > 2 * 16 * cu_count())
        return run_stream<AR, 2, 4, D2, EPI_STORE>(A, lda, B, ldb, M, N, K, epi, s);
      return run_stream<AR, 1, 8, D1, EPI_STORE>(A, lda, B, ldb, M, N, K, epi, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_stream(const void* A, int lda, const void* B, int ldb, int M, int N, int K,
                         const Epi& epi, hipStream_t s) {
  if (M == 0) return hipSuccess;
  if (M > kStreamMaxRows) return hipErrorInvalidValue;
  if (M <= 8) return stream_rows<8>(A, lda, B, ldb, M, N, K, epi, s);
  return stream_rows<16>(A, lda, B, ldb, M, N, K, epi, s);
}

bool stream_norm_ok(int M, int K) {
  return M <= 8 && K <= kStreamNormMaxCols && M * K <= kStreamNormMaxElems;
}

hipError_t launch_stream_norm_swiglu(const void* x, int ldx, const void* B, int ldb, int M, int K,
                                     const Epi& epi, const StreamNorm& nrm, hipStream_t s) {
  if (M == 0) return hipSuccess;
  if (!stream_norm_ok(M, K)) return hipErrorInvalidValue;
  return run_stream<8, 2, 4, 4, EPI_SWIGLU, true>(x, ldx, B, ldb, M, 2 * epi.ffn, K, epi, s, nrm);
}

}  // namespace tri
