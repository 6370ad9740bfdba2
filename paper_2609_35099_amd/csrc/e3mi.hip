// e3mi: channelwise Clebsch-Gordan tensor product and message-passing
// convolution for MI355X (gfx950).  Kernels and the C ABI declared in
// include/e3mi.h.
//
// Execution model (the same for every kernel that touches features):
//   * lanes = channels.  A 64-lane wave covers C channels with CPL = C/64
//     consecutive channels per lane, so every feature row (C floats) is one
//     coalesced vector load or store; the feature axis is walked in registers.
//   * per edge (or tensor-product row), the channel-independent
//     pre-contraction A[(path, M), m1] = sum_m2 C[M, m1, m2] y[m2] (records
//     grouped by output then x coordinate, App. E.4's MessageTile grouping) is
//     computed once with lane = edge and staged in LDS; the per-channel loop
//     reads it back as wave-uniform broadcasts.  The coupling constants are
//     compile-time literals (generated per irreps variant).
//   * a wave owns one receiver and one group of paths (forward) or one group
//     of whole x blocks (backward); its accumulators live in registers and are
//     stored once (App. E.3 receiver-stationary aggregation).  No atomics.
//   * workgroups are single waves; block ids are mapped so that each XCD
//     walks a contiguous range of receivers and the groups of one receiver run
//     back to back on the same XCD (shared L2 for the sender gathers).

#include "e3mi_impl.h"

// ------------------------------------------------------------ shared state
thread_local std::string g_last_error;
Timing g_timing;

// The compiled variants, each defined in its own unit (generated list).
#include "generated/variant_table.inc"

namespace {
// ------------------------------------------------------------ linear mixing
// Dense per-irrep channel mixing on the matrix cores (float32 in and out; the
// kernels are in linear_split.h).  A destination block of 2l+1 rows per node
// receives, for each of its sources, src[n, src_row + m, k] B[k, col] summed
// over k and the sources.  The forward has one job per output block (its
// sources: the input blocks of the same degree and parity; B = W); dx has one
// job per input block (its sources: the output blocks it feeds; B = W
// transposed).
constexpr int kLinMaxJobs = 64;
constexpr int kLinChunks = 64;  // row chunks of the dW reduction (fixed: deterministic)

struct LinJob {
  int R, dst_row, src_first, nsrc;
};
struct LinSrc {
  int row, pad;
  int64_t w_off;
};
struct LinPair {  // dW slice: input block row, output block row, W offset
  int R, src_row, dst_row, pad;
  int64_t w_off;
};

struct LinArgs {
  const float* src;
  const float* W;
  float* dst;
  const LinJob* jobs;
  const LinSrc* srcs;
  int64_t n;
  int D_src, C_src, D_dst, C_dst, njobs, slabs;
  int first[kLinMaxJobs + 1];
};

// Wt[pair][j][k] = W[w_off(pair) + k C_out + j]: each dW-sized slice
// transposed, for a dx whose W is not 16-byte aligned.
__global__ __launch_bounds__(256) void k_lin_transpose(const float* __restrict__ W, const LinPair* __restrict__ pairs,
                                                        float* __restrict__ Wt, int npairs, int C_in, int C_out) {
  const int64_t per = (int64_t)C_in * C_out;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= per * npairs) return;
  const int p = (int)(i / per);
  const int64_t e = i % per;
  const int j = (int)(e / C_in), k = (int)(e % C_in);
  Wt[i] = W[pairs[p].w_off + (int64_t)k * C_out + j];
}

struct LinDwArgs {
  const float* x;
  const float* dout;
  float* dWp;  // [npairs][kLinChunks][C_in][C_out]
  const LinPair* pairs;
  int64_t n;
  int D_in, C_in, D_out, C_out, ktiles, jtiles, npairs;
};

// dW[w_off(p) + e] = sum over the row chunks of pair p, in chunk order.
__global__ __launch_bounds__(256) void k_lin_dw_sum(const float* __restrict__ dWp, const LinPair* __restrict__ pairs,
                                                     float* __restrict__ dW, int npairs, int64_t per) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)npairs * per) return;
  const int p = (int)(i / per);
  const int64_t e = i % per;
  float s = 0.0f;
  for (int c = 0; c < kLinChunks; ++c) s += dWp[((int64_t)p * kLinChunks + c) * per + e];
  dW[pairs[p].w_off + e] = s;
}

}  // namespace
#include "linear_split.h"
namespace {

// ------------------------------------------------------------ generic records
// Tensor product with caller-supplied records (App. E.2's unfolded form):
//   out[r, o, q] = sum over the records of segment o of v A[r, a, q] B[r, b, (q)]
// Rows and channels are independent, so a wave takes RB x 64 consecutive
// (row, channel) pairs, whatever C is (64-channel slabs of a row left lanes
// idle at any other C, and shared cache lines between waves of different XCDs
// at C = 100).  The operands are staged in LDS as [a][u][lane] (pair 64 u +
// lane, so one address serves the RB pairs of a lane); each record feeds RB
// fused multiply-adds.  The backward is the same kernel on permuted record
// tables (eq. tp-bwd).  With RED the outputs are summed over the channels (a
// shared y's cotangent): a wave takes whole rows, or one piece of a row longer
// than RB x 64 (its partials then added by k_tpg_sum), and adds in a fixed
// order.
//
// What bounds it is latency and instruction issue, not the LDS reads (38% of
// their rate), so nothing in the chain waits alone: the float32 operands go
// straight to LDS with every load in flight at once; a chunk of 64 records is
// one coalesced load, a record per lane, handed out by v_readlane (scalar loads
// would share the LDS reads' wait counter), and the next chunk's is in flight;
// the operands of the next AH records are read while the current ones are used,
// and a group of records in which no segment ends takes no branches.  Per
// kernel, against scalar records, rows of four and slabs of 64 channels: 9 + 9
// operand rows and 137 records (30,011 rows, C = 100) 189 -> 111 us; 16 + 16
// rows, 611 records (20,000 rows, C = 64) 303 -> 210 us; 16 records (50,000 rows,
// C = 128) 63 -> 58 us.  A shared B, staged per channel as well at first, had
// lost to that (9 + 16 rows, 100,000 rows, C = 128: forward 531, then 663 us, dx
// 707, then 1053); staged once it takes 562 and 680 us, and with 9 + 9 rows
// (50,000 rows, C = 128) 135 and 136 us against 148 and 152.
constexpr int kTpgAhead = 8;

// A segment's last record carries kTpgEnd; a segment without records has one
// with kTpgEmpty, which stores zeros.  Tables are padded to a multiple of
// kTpgAhead with records that belong to no segment.
constexpr unsigned kTpgEnd = 1u << 30, kTpgEmpty = 1u << 31;
struct TpgRec {
  unsigned ab;  // a | b << 10 | flags (operand rows: at most 256 fit the staging)
  float v;
};
struct TpgRec64 {
  unsigned ab;
  unsigned pad;
  double v;
};
template <class T>
struct TpgArgs {
  const T* A;
  const T* B;
  T* out;
  T* part;  // RED: [rows][pieces][dout] (dy itself when pieces == 1)
  const typename std::conditional<sizeof(T) == 8, TpgRec64, TpgRec>::type* recs;
  int nrec;
  int64_t rows;
  int C, dA, dB, dout;
  int pieces;  // RED: tiles of one row (1: `rpt` whole rows per tile)
  int rpt;
};

__device__ __forceinline__ float lane_of(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_of(double v, int l) {
  const uint64_t x = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)x, l);
  const unsigned hi = __builtin_amdgcn_readlane((int)(unsigned)(x >> 32), l);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Rows that `pairs` consecutive (row, channel) pairs can touch.
__host__ __device__ inline int tpg_tile_rows(int C, int pairs) { return (C + pairs - 2) / C + 1; }

template <class T>
__device__ __forceinline__ T buf_ld(__amdgpu_buffer_rsrc_t r, int off, int soff) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}

// B: one value per (row, channel); or shared by the channels of a row and
// staged per row of the tile, each lane with its own row's address; or shared
// and staged per 64 pairs (C % 64 == 0, where they lie in one row), the values
// of a lane's pairs side by side.
enum TpgB { kTpgBOwn, kTpgBRow, kTpgBOnce };

// AH: records whose operands are read ahead (4 or kTpgAhead).
template <class T, int BM, bool RED, int RB, int AH>
__global__ __launch_bounds__(kWave) void k_tpg(TpgArgs<T> a) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T* sA = reinterpret_cast<T*>(lds_raw);     // [dA][RB][64]
  constexpr bool BSH = BM != kTpgBOwn;
  T* sB = sA + a.dA * RB * kWave;            // [dB][RB][64], kTpgBRow: [rows][dB | 1], kTpgBOnce: [dB][RB]
  T* sP = sB + a.dB * RB * kWave;            // RED (own B): [dout][RB][64]
  const int lane = threadIdx.x, C = a.C;
  constexpr int kPairs = RB * kWave;
  // first row and channel of the tile, and its number of pairs
  const int64_t tile = block_id();
  int64_t r0;
  int c0, np;
  if constexpr (RED) {
    r0 = a.pieces == 1 ? tile * a.rpt : tile / a.pieces;
    if (r0 >= a.rows) return;
    c0 = a.pieces == 1 ? 0 : (int)(tile % a.pieces) * kPairs;
    np = a.pieces == 1 ? (int)(a.rows - r0 < a.rpt ? a.rows - r0 : a.rpt) * C : imin(kPairs, C - c0);
  } else {
    const int64_t p0 = tile * kPairs, left = a.rows * C - p0;
    if (left <= 0) return;
    r0 = p0 / C, c0 = (int)(p0 - r0 * C);
    np = left < kPairs ? (int)left : kPairs;
  }
  // the lane's pairs: row r0 + dr, channel q; operand offsets from row r0
  unsigned offA[RB], offB[RB];
  int rowB[RB];  // kTpgBRow: the pair's row in sB
  T* po[RB];
#pragma unroll
  for (int u = 0; u < RB; ++u) {
    const int i = u * kWave + lane, at = c0 + i, dr = at / C, q = at - dr * C;
    const bool on = i < np;
    offA[u] = on ? (unsigned)(dr * a.dA * C + q) * (unsigned)sizeof(T) : kSubOff;
    offB[u] = on ? (unsigned)(dr * a.dB * C + q) * (unsigned)sizeof(T) : kSubOff;
    rowB[u] = dr * (a.dB | 1);
    po[u] = a.out + ((r0 + dr) * a.dout * C + q);
  }
  auto rsrc = [&](const T* p, int64_t row) {
    const int64_t n = (a.rows - r0) * row * (int64_t)sizeof(T);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p) + r0 * row, (short)0,
                                             (int)(unsigned)(n < (int64_t)kSubOff ? n : (int64_t)kSubOff), 0x00020000);
  };
  auto stage = [&](__amdgpu_buffer_rsrc_t r, T* dst, int d, const unsigned (&off)[RB], int stride) {
    if constexpr (sizeof(T) == 4) {
      for (int ai = 0; ai < d; ++ai)
#pragma unroll
        for (int u = 0; u < RB; ++u)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              r, (__attribute__((address_space(3))) void*)(dst + (ai * RB + u) * kWave), 4, (int)off[u],
              ai * stride * 4, 0, 0);
    } else {
      constexpr int N = (RED ? 16 : 32) / RB;  // operand rows in flight
      auto rows = [&](auto n, int a0) {
        constexpr int N = decltype(n)::value;
        T v[N][RB];
#pragma unroll
        for (int k = 0; k < N; ++k)
#pragma unroll
          for (int u = 0; u < RB; ++u)
            v[k][u] = buf_ld<T>(r, a0 + k < d ? (int)off[u] : (int)kSubOff, (a0 + k) * stride * (int)sizeof(T));
#pragma unroll
        for (int k = 0; k < N; ++k)
          if (a0 + k < d)
#pragma unroll
            for (int u = 0; u < RB; ++u) dst[((a0 + k) * RB + u) * kWave + lane] = v[k][u];
      };
      // a remainder takes no more requests than the next power of two (one operand
      // row, 22,137 rows of 128 channels: 17.7 -> 14.1 us)
      int a0 = 0;
      for (; d - a0 > N / 2; a0 += N) rows(std::integral_constant<int, N>{}, a0);
      const int left = d - a0;
      if (left > N / 4)
        rows(std::integral_constant<int, N / 2>{}, a0);
      else if (left > N / 8)
        rows(std::integral_constant<int, N / 4>{}, a0);
      else if (left > 0)
        rows(std::integral_constant<int, (N < 8 ? 1 : N / 8)>{}, a0);
    }
  };
  // The first records are requested before the operands, and a shared B of
  // float64, which goes through registers, before A: neither waits for the other
  // (float64, 4 + 4 rows, 12,500 rows of 128 channels: 25 -> 22 us; float32, 9 +
  // 16 rows, 100,000 rows of 128: dx 702 -> 680 us).
  constexpr bool kBFirst = BM != kTpgBOwn && sizeof(T) == 8;
  const auto record = [&](int k0) { return a.recs[k0 + imin(lane, imin(kWave, a.nrec - k0) - 1)]; };
  auto next = record(0);
  if constexpr (!kBFirst) stage(rsrc(a.A, (int64_t)a.dA * C), sA, a.dA, offA, C);
  const __amdgpu_buffer_rsrc_t brsrc = rsrc(a.B, (int64_t)a.dB * (BSH ? 1 : C));
  if constexpr (BM == kTpgBOnce) {
    for (int i = lane; i < a.dB * RB; i += kWave) {
      const int dr = (c0 + (i % RB) * kWave) / C;  // past the last row: reads zero
      sB[i] = buf_ld<T>(brsrc, (dr * a.dB + i / RB) * (int)sizeof(T), 0);
    }
  } else if constexpr (BM == kTpgBRow) {
    const SpDiv div(a.dB);
#pragma unroll 4
    for (int i = lane; i < tpg_tile_rows(C, kPairs) * a.dB; i += kWave) {
      int b;
      const int dr = div(i, b);
      sB[dr * (a.dB | 1) + b] = buf_ld<T>(brsrc, i * (int)sizeof(T), 0);  // past the last row: zero
    }
  } else {
    stage(brsrc, sB, a.dB, offB, C);
  }
  if constexpr (kBFirst) stage(rsrc(a.A, (int64_t)a.dA * C), sA, a.dA, offA, C);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads to LDS
  __syncthreads();
  int o = 0;
  T acc[RB];
#pragma unroll
  for (int u = 0; u < RB; ++u) acc[u] = T(0);
  for (int k0 = 0; k0 < a.nrec; k0 += kWave) {
    const int nk = imin(kWave, a.nrec - k0);  // a multiple of kTpgAhead
    const auto mine = next;
    if (k0 + kWave < a.nrec) next = record(k0 + kWave);
    const T my_v = T(mine.v);
    // per lane: LDS offsets of its record's operands; per chunk: the flag bits
    const int my_a = (int)(mine.ab & 0x3ffu) * (RB * kWave);
    const int my_b = (int)(mine.ab >> 10 & 0x3ffu) * (BM == kTpgBOwn ? RB * kWave : BM == kTpgBOnce ? RB : 1);
    const uint64_t ends = __ballot((mine.ab & (kTpgEnd | kTpgEmpty)) != 0), empties = __ballot((mine.ab & kTpgEmpty) != 0);
    T pa[2][AH][RB], pb[2][AH][RB];
    auto fetch = [&](int k, T (&va)[AH][RB], T (&vb)[AH][RB]) {
#pragma unroll
      for (int j = 0; j < AH; ++j) {
        const T* qa = sA + __builtin_amdgcn_readlane(my_a, k + j) + lane;
        const T* qb = sB + __builtin_amdgcn_readlane(my_b, k + j);
#pragma unroll
        for (int u = 0; u < RB; ++u) va[j][u] = qa[u * kWave];
        if constexpr (BM == kTpgBOnce && RB > 1) {
          typedef T Bv __attribute__((ext_vector_type(RB)));
          const Bv b = *reinterpret_cast<const Bv*>(qb);
#pragma unroll
          for (int u = 0; u < RB; ++u) vb[j][u] = b[u];
        } else {
#pragma unroll
          for (int u = 0; u < RB; ++u) vb[j][u] = qb[BM == kTpgBOwn ? u * kWave + lane : BM == kTpgBRow ? rowB[u] : 0];
        }
      }
    };
    auto use = [&](int k, const T (&va)[AH][RB], const T (&vb)[AH][RB]) {
      const unsigned end = (unsigned)(ends >> k) & ((1u << AH) - 1), empty = (unsigned)(empties >> k);
      if (end == 0) {  // most groups: no segment ends inside
#pragma unroll
        for (int j = 0; j < AH; ++j) {
          const T rv = lane_of(my_v, k + j);
#pragma unroll
          for (int u = 0; u < RB; ++u) acc[u] = fma(rv * va[j][u], vb[j][u], acc[u]);
        }
        return;
      }
#pragma unroll
      for (int j = 0; j < AH; ++j) {
        const T rv = lane_of(my_v, k + j);
#pragma unroll
        for (int u = 0; u < RB; ++u) acc[u] = fma(rv * va[j][u], vb[j][u], acc[u]);
        if (end >> j & 1) {
          if (empty >> j & 1) {
#pragma unroll
            for (int u = 0; u < RB; ++u) acc[u] = T(0);
          }
          if constexpr (RED) {
#pragma unroll
            for (int u = 0; u < RB; ++u) sP[(o * RB + u) * kWave + lane] = acc[u];
          } else {
            const int64_t at = (int64_t)o * C;
#pragma unroll
            for (int u = 0; u < RB; ++u)
              if (u * kWave + lane < np) po[u][at] = acc[u];
          }
#pragma unroll
          for (int u = 0; u < RB; ++u) acc[u] = T(0);
          ++o;
        }
      }
    };
    fetch(0, pa[0], pb[0]);
    for (int k = 0; k < nk; k += 2 * AH) {
      if (k + AH < nk) fetch(k + AH, pa[1], pb[1]);
      use(k, pa[0], pb[0]);
      if (k + AH < nk) {
        if (k + 2 * AH < nk) fetch(k + 2 * AH, pa[0], pb[0]);
        use(k + AH, pa[1], pb[1]);
      }
    }
  }
  if constexpr (RED) {
    __syncthreads();
    const int w = a.pieces == 1 ? C : np, nrow = np / w;  // channels and rows of the tile
    // runs of at most 64 channels, a lane each (longer chains round larger sums:
    // float32, 256 channels of one sign, 3.2 times the error), then a row's runs
    const int nrun = (w + kWave - 1) / kWave;
    for (int i = lane; i < a.dout * nrow * nrun; i += kWave) {
      const int run = i % nrun, our = i / nrun, ou = our / nrow, r = our - ou * nrow;
      T* p = sP + ou * kPairs + r * w + run * kWave;
      const int n = imin(kWave, w - run * kWave);
      T t = T(0);
      // lane i starts at another channel, so that the lanes read different banks
      constexpr int W = 16 / sizeof(T);
      if (n == kWave && w % W == 0) {
        // reads of 16 bytes whose addresses do not wait for one another (22,137 rows
        // of 128 channels, 4 + 4 operand rows, 9 records: backward 46 -> 41 us)
        typedef T Tv __attribute__((ext_vector_type(W)));
#pragma unroll
        for (int l = 0; l < kWave / W; ++l) {
          const Tv v = reinterpret_cast<const Tv*>(p)[(l + i) % (kWave / W)];
#pragma unroll
          for (int k = 0; k < W; ++k) t += v[k];
        }
      } else {
#pragma unroll 4
        for (int l = 0, c = i % n; l < n; ++l) {
          t += p[c];
          c = c + 1 == n ? 0 : c + 1;
        }
      }
      p[0] = t;
    }
    __syncthreads();
    for (int i = lane; i < a.dout * nrow; i += kWave) {
      const int ou = i / nrow, r = i - ou * nrow;
      const T* p = sP + ou * kPairs + r * w;
      T t = p[0];
      for (int run = 1; run < nrun; ++run) t += p[run * kWave];
      a.part[((r0 + r) * a.pieces + (a.pieces == 1 ? 0 : tile % a.pieces)) * a.dout + ou] = t;
    }
  }
}

template <class T>
__global__ __launch_bounds__(256) void k_tpg_sum(const T* __restrict__ part, T* __restrict__ out, int64_t rows,
                                                  int nslab, int dout) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * dout) return;
  const int64_t r = i / dout;
  const int o = (int)(i % dout);
  T t = T(0);
  for (int sl = 0; sl < nslab; ++sl) t += part[(r * nslab + sl) * dout + o];
  out[i] = t;
}

// ------------------------------------------------------------ graph
__global__ void k_graph_keys(const int32_t* __restrict__ snd, const int32_t* __restrict__ rcv, int64_t n_edges,
                             int32_t n_nodes, int32_t pad, uint32_t* __restrict__ key_r, uint32_t* __restrict__ key_s,
                             int* __restrict__ bad) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n_edges) return;
  const int32_t s = snd[e], r = rcv[e];
  const bool out_of_range = s < 0 || s >= n_nodes || r < 0 || r >= n_nodes;
  if (out_of_range) *bad = 1;  // every writer stores the same value
  // an out-of-range index becomes the padding key (the build fails anyway),
  // so that the sort's digits stay below 2^bits
  const bool is_pad = out_of_range || (pad >= 0 && (s == pad || r == pad));
  key_r[e] = is_pad ? (uint32_t)n_nodes : (uint32_t)r;
  key_s[e] = is_pad ? (uint32_t)n_nodes : (uint32_t)s;
}

// Stable LSD radix sort of (key, edge id) pairs, 8 bits of the key per pass.
// A tile is kSortRounds rounds of one 256-thread block over consecutive
// elements.  Per pass: k_sort_hist counts each tile's digits, k_sort_scan turns
// each digit's tile counts into exclusive offsets and a digit total, and
// k_sort_scatter places every element at
//   (elements of smaller digits) + offset[digit][tile]
//   + (same-digit elements of earlier rounds of its tile)
//   + (same-digit elements of earlier waves of its round)
//   + (same-digit elements of lower lanes of its wave),
// so equal digits keep their input order and every pass is stable.  Integer
// counts only: the result does not depend on scheduling.
//
// The receiver and the sender sort run in the same launches (blockIdx.y).  A
// tile has 4 rounds up to kSortLarge elements, where its rounds are a serial
// chain in a launch that does not fill the chip, and 16 beyond, where shorter
// tiles would lengthen the scan (build and destruction with 4 and 16 rounds: 116 and
// 141 us at 87,000 edges, 213 and 229 at 320,000, 286 and 271 at 900,000, 338 and 317
// at 1,270,000).
constexpr int kSortBlock = 256;
constexpr int64_t kSortLarge = 1 << 19;
inline int64_t sort_tiles(int64_t n) {
  const int64_t tile = (int64_t)kSortBlock * (n <= kSortLarge ? 4 : 16);
  return (n + tile - 1) / tile;
}
constexpr int kSortWaves = kSortBlock / kWave;
static_assert(kSortBlock == 256, "one thread per digit");

// One pass of the two sorts; iin == nullptr: the ids are the element indices.
// count: 256 x tiles tile counts, then 256 digit totals.
struct SortPass {
  const uint32_t* kin[2];
  const int32_t* iin[2];
  uint32_t* kout[2];
  int32_t* iout[2];
  int32_t* count[2];
};

template <int ROUNDS>
__global__ __launch_bounds__(kSortBlock) void k_sort_hist(SortPass a, int64_t n, int shift, int64_t n_tiles) {
  constexpr int kSortRounds = ROUNDS, kSortTile = kSortBlock * ROUNDS;
  __shared__ int hist[256];
  const uint32_t* __restrict__ keys = a.kin[blockIdx.y];
  int32_t* __restrict__ count = a.count[blockIdx.y];
  const int tid = threadIdx.x;
  hist[tid] = 0;
  __syncthreads();
  const int64_t t = blockIdx.x;
  for (int j = 0; j < kSortRounds; ++j) {
    const int64_t i = t * kSortTile + (int64_t)j * kSortBlock + tid;
    if (i < n) atomicAdd(&hist[(keys[i] >> shift) & 255u], 1);
  }
  __syncthreads();
  count[(int64_t)tid * n_tiles + t] = hist[tid];
}

// Inclusive scan of v over the block (Hillis-Steele in LDS); total = the sum
// over the block.  Ends with a barrier after the last reads of buf.
__device__ __forceinline__ int32_t block_incl_scan(int32_t v, int32_t (&buf)[2][kSortBlock], int tid,
                                                   int32_t& total) {
  buf[0][tid] = v;
  __syncthreads();
  int cur = 0;
  for (int d = 1; d < kSortBlock; d <<= 1) {
    const int32_t u = buf[cur][tid] + (tid >= d ? buf[cur][tid - d] : 0);
    buf[cur ^ 1][tid] = u;
    cur ^= 1;
    __syncthreads();
  }
  const int32_t incl = buf[cur][tid];
  total = buf[cur][kSortBlock - 1];
  __syncthreads();
  return incl;
}

// Per digit (one block each): exclusive scan of its tiles' counts in place
// (row d of count) and the digit's total.
__global__ __launch_bounds__(kSortBlock) void k_sort_scan(SortPass a, int64_t n_tiles) {
  __shared__ int32_t buf[2][kSortBlock];
  int32_t *count = a.count[blockIdx.y], *total = count + 256 * n_tiles;
  const int tid = threadIdx.x;
  int32_t* row = count + (int64_t)blockIdx.x * n_tiles;
  int32_t carry = 0;
  for (int64_t c0 = 0; c0 < n_tiles; c0 += kSortBlock) {
    const int64_t i = c0 + tid;
    const int32_t v = i < n_tiles ? row[i] : 0;
    int32_t chunk = 0;
    const int32_t incl = block_incl_scan(v, buf, tid, chunk);
    if (i < n_tiles) row[i] = carry + incl - v;
    carry += chunk;
  }
  if (tid == 0) total[blockIdx.x] = carry;
}

// Positions outside [0, n) cannot arise from consistent offsets; they are
// refused (bad = 1) rather than written.
template <int ROUNDS>
__global__ __launch_bounds__(kSortBlock) void k_sort_scatter(SortPass a, int64_t n, int shift, int64_t n_tiles,
                                                             int* __restrict__ bad) {
  constexpr int kSortRounds = ROUNDS, kSortTile = kSortBlock * ROUNDS;
  const uint32_t* __restrict__ keys_in = a.kin[blockIdx.y];
  const int32_t* __restrict__ ids_in = a.iin[blockIdx.y];
  const int32_t* __restrict__ off = a.count[blockIdx.y];
  const int32_t* __restrict__ total = off + 256 * n_tiles;
  uint32_t* __restrict__ keys_out = a.kout[blockIdx.y];
  int32_t* __restrict__ ids_out = a.iout[blockIdx.y];
  __shared__ int running[256];
  __shared__ int cnt[kSortWaves][256];
  __shared__ int32_t buf[2][kSortBlock];
  const int tid = threadIdx.x, lane = tid % kWave, w = tid / kWave;
  {
    // running starts at the digit's base: the elements of all smaller digits
    int32_t all = 0;
    const int32_t v = total[tid];
    running[tid] = block_incl_scan(v, buf, tid, all) - v;
  }
#pragma unroll
  for (int k = 0; k < kSortWaves; ++k) cnt[k][tid] = 0;
  __syncthreads();
  const int64_t t = blockIdx.x;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (kWave - lane));
  for (int j = 0; j < kSortRounds; ++j) {
    const int64_t i = t * kSortTile + (int64_t)j * kSortBlock + tid;
    const bool valid = i < n;
    const uint32_t key = valid ? keys_in[i] : 0u;
    const int32_t id = valid ? (ids_in ? ids_in[i] : (int32_t)i) : 0;
    const int d = (int)((key >> shift) & 255u);
    // lanes of this wave holding the same digit
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) {
      const uint64_t set = __ballot(valid && ((d >> bit) & 1));
      same &= ((d >> bit) & 1) ? set : ~set;
    }
    const int rank = __popcll(same & below);
    if (valid && (same & below) == 0) cnt[w][d] = __popcll(same);  // the digit's lowest lane
    __syncthreads();
    if (valid) {
      int prefix = 0;
      for (int k = 0; k < w; ++k) prefix += cnt[k][d];
      const int64_t pos = (int64_t)off[(int64_t)d * n_tiles + t] + running[d] + prefix + rank;
      if (pos >= 0 && pos < n) {
        keys_out[pos] = key;
        ids_out[pos] = id;
      } else {
        *bad = 1;
      }
    }
    __syncthreads();
    int add = 0;
#pragma unroll
    for (int k = 0; k < kSortWaves; ++k) add += cnt[k][tid], cnt[k][tid] = 0;
    running[tid] += add;
    __syncthreads();
  }
}

// rowptr[b] = first position with key >= b (binary search; keys sorted), for
// both sorts; the receiver one also reports the live edges, rowptr[n_nodes].
__global__ void k_graph_rowptr(const uint32_t* __restrict__ keys_r, const uint32_t* __restrict__ keys_s,
                               int64_t n_edges, int32_t n_nodes, int32_t* __restrict__ rowptr_r,
                               int32_t* __restrict__ rowptr_s, int* __restrict__ n_live) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b > n_nodes) return;
  const uint32_t* keys = blockIdx.y ? keys_s : keys_r;
  int64_t lo = 0, hi = n_edges;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (keys[mid] < (uint32_t)b)
      lo = mid + 1;
    else
      hi = mid;
  }
  (blockIdx.y ? rowptr_s : rowptr_r)[b] = (int32_t)lo;
  if (blockIdx.y == 0 && b == n_nodes) *n_live = (int)lo;
}

// flag: index out of range, inconsistent offsets (the ids are then not
// followed), live edges.
__global__ void k_graph_finish(const int32_t* __restrict__ snd, const int32_t* __restrict__ eid_r,
                               const int32_t* __restrict__ eid_s, const int* __restrict__ flag,
                               int32_t* __restrict__ src_r, int32_t* __restrict__ pos_s) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (flag[1] || i >= flag[2]) return;
  src_r[i] = snd[eid_r[i]];
  pos_s[eid_s[i]] = (int32_t)i;
}

__global__ void k_graph_r2s(const int32_t* __restrict__ eid_r, const int32_t* __restrict__ pos_s,
                            const int* __restrict__ flag, int32_t* __restrict__ r2s) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (flag[1] || i >= flag[2]) return;
  r2s[i] = pos_s[eid_r[i]];
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// A compiled variant (every entry point).
e3_status check_plan(const e3_plan* p) {
  if (!p) return E3_ERR_INVALID_ARG;
  if (p->variant < 0) {
    g_last_error = p->rec ? "this entry point needs a compiled kernel variant for the layout"
                          : p->no_rec_reason;
    return E3_ERR_UNSUPPORTED;
  }
  return E3_OK;
}

// A compiled variant, or the record path with its tables on the current
// device (the convolution and tensor-product forward and backward).
e3_status check_any(const e3_plan* p) {
  if (!p) return E3_ERR_INVALID_ARG;
  return p->variant >= 0 ? E3_OK : rec_check(p);
}

// A compiled variant or the composed path (the float64 builds and the fused
// radial weights, which the record path does not have).
e3_status check_composable(const e3_plan* p) {
  if (!p) return E3_ERR_INVALID_ARG;
  if (p->variant >= 0 || p->composed) return E3_OK;
  g_last_error = p->rec ? "this entry point needs a compiled variant or the composed path" : p->no_rec_reason;
  return E3_ERR_UNSUPPORTED;
}

Ws conv_ws(const e3_plan* p, const e3_graph* g) {
  return p->variant >= 0 ? (*kVariants[p->variant]()).ws(p, g) : rec_ws(p, g);
}
}  // namespace


// ============================================================ C ABI
extern "C" {

const char* e3_status_str(e3_status s) {
  switch (s) {
    case E3_OK: return "ok";
    case E3_ERR_INVALID_ARG: return "invalid argument";
    case E3_ERR_UNSUPPORTED: return "unsupported configuration";
    case E3_ERR_INDEX_OUT_OF_RANGE: return "edge index out of range";
    case E3_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
    case E3_ERR_HIP: return "HIP runtime error";
    case E3_ERR_ALLOC: return "allocation failed";
  }
  return "unknown status";
}

const char* e3_last_error(void) { return g_last_error.c_str(); }

e3_status e3_timing_enable(int on) {
  std::lock_guard<std::mutex> lk(g_timing.mu);
  g_timing.on = on != 0;
  return E3_OK;
}

e3_status e3_timing_reset(void) {
  std::lock_guard<std::mutex> lk(g_timing.mu);
  for (auto& p : g_timing.pending) {
    (void)hipEventSynchronize(p.b);
    g_timing.pool.push_back(p.a);
    g_timing.pool.push_back(p.b);
  }
  g_timing.pending.clear();
  g_timing.acc.clear();
  return E3_OK;
}

e3_status e3_timing_read(int cap, char* names, double* ms, int64_t* count, int* n) {
  if (cap < 0 || !n || (cap > 0 && (!names || !ms || !count))) return E3_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(g_timing.mu);
  for (auto& p : g_timing.pending) {
    E3_HIP(hipEventSynchronize(p.b));
    float t = 0.0f;
    E3_HIP(hipEventElapsedTime(&t, p.a, p.b));
    auto& slot = g_timing.acc[p.name];
    slot.first += t;
    slot.second += 1;
    g_timing.pool.push_back(p.a);
    g_timing.pool.push_back(p.b);
  }
  g_timing.pending.clear();
  int i = 0;
  for (const auto& [name, v] : g_timing.acc) {
    if (i < cap) {
      std::memset(names + 32 * i, 0, 32);
      std::strncpy(names + 32 * i, name.c_str(), 31);
      ms[i] = v.first;
      count[i] = v.second;
    }
    ++i;
  }
  *n = i;
  return E3_OK;
}

e3_status e3_plan_create(const char* irreps_x, int lmax_sh, int lmax_out, unsigned flags, e3_plan** out) {
  if (!irreps_x || !out) return E3_ERR_INVALID_ARG;
  *out = nullptr;
  if (lmax_sh < 0 || lmax_sh > 3 || lmax_out < 0 || lmax_out > 16 ||
      (flags & ~(E3_PARITY_NATURAL | E3_PLAN_RECORDS | E3_PLAN_COMPOSED)) ||
      ((flags & E3_PLAN_RECORDS) && (flags & E3_PLAN_COMPOSED)))
    return E3_ERR_INVALID_ARG;
  std::vector<e3b::Block> blocks;
  std::string err;
  if (!e3b::parse_irreps(irreps_x, blocks, err)) {
    g_last_error = err;
    return E3_ERR_INVALID_ARG;
  }
  for (const auto& b : blocks)
    if (b.l > 16) return E3_ERR_INVALID_ARG;
  e3_plan* p = new (std::nothrow) e3_plan();
  if (!p) return E3_ERR_ALLOC;
  if (!e3b::make_layout(irreps_x, lmax_sh, lmax_out, (flags & E3_PARITY_NATURAL) != 0, p->lay, err)) {
    g_last_error = err;
    delete p;
    return E3_ERR_UNSUPPORTED;
  }
  try {
    p->recs = e3b::coo(p->lay);
  } catch (const std::exception& ex) {
    g_last_error = ex.what();
    delete p;
    return E3_ERR_UNSUPPORTED;
  }
  const std::string sig = e3b::path_signature(p->lay);
  // Channels: multiples of 4 up to kMaxChannels.  The forward, tensor-product
  // and dx kernels give each lane 2 consecutive channels when C > 64 (one lane
  // per channel otherwise); the backward sweep gives each lane 1.  Channels
  // beyond one wave are covered by further 64-lane slabs.
  const int C = p->lay.C;
  if (C >= 4 && C % 4 == 0 && C <= kMaxChannels && !(flags & (E3_PLAN_RECORDS | E3_PLAN_COMPOSED))) {
    for (int i = 0; i < kNumVariants; ++i)
      if (sig == kVariants[i]()->sig && p->lay.d_sh == kVariants[i]()->d_sh) p->variant = i;
  }
  if (p->variant >= 0) {
    p->cpl_f = C <= kWave ? 1 : E3_FWD_CPL;
    p->nslab_f = (C + kWave * p->cpl_f - 1) / (kWave * p->cpl_f);
    p->nslab_b = (C + kWave - 1) / kWave;
  } else if ((flags & E3_PLAN_RECORDS) || comp_create(p) != E3_OK) {
    // still a valid plan (its tables can be queried) when neither path takes
    // it: its compute calls report why
    if (flags & E3_PLAN_COMPOSED)
      p->no_rec_reason = "the composed path takes x blocks and outputs of degree <= 3 and C a multiple of 4 "
                         "up to " + std::to_string(kMaxChannels);
    else if (rec_create(p) != E3_OK)
      p->no_rec_reason = g_last_error;
  }
  *out = p;
  return E3_OK;
}

e3_status e3_plan_query(const e3_plan* p, e3_plan_info* info) {
  if (!p || !info) return E3_ERR_INVALID_ARG;
  info->C = p->lay.C;
  info->P = (int)p->lay.paths.size();
  info->D_in = p->lay.d_in;
  info->D_sh = p->lay.d_sh;
  info->D_out = p->lay.d_out;
  info->nnz = (int)p->recs.size();
  info->lmax_sh = p->lay.lmax_sh;
  info->lmax_out = p->lay.lmax_out;
  info->supported = p->variant >= 0 ? 1 : p->composed ? 3 : (rec_ready(p) ? 2 : 0);
  return E3_OK;
}

e3_status e3_plan_destroy(e3_plan* p) {
  delete p;
  return E3_OK;
}

e3_status e3_plan_paths(const e3_plan* p, int32_t* out) {
  if (!p || !out) return E3_ERR_INVALID_ARG;
  for (size_t i = 0; i < p->lay.paths.size(); ++i) {
    const auto& q = p->lay.paths[i];
    const int32_t v[7] = {q.l1, q.l2, q.l3, q.p3, q.x_off, q.y_off, q.out_off};
    std::memcpy(out + 7 * i, v, sizeof(v));
  }
  return E3_OK;
}

e3_status e3_plan_records(const e3_plan* p, int64_t cap, int32_t* i0, int32_t* i1, int32_t* i2, double* val,
                          int64_t* n) {
  if (!p || !n || cap < 0) return E3_ERR_INVALID_ARG;
  *n = (int64_t)p->recs.size();
  const int64_t m = std::min<int64_t>(cap, *n);
  if (m > 0 && (!i0 || !i1 || !i2 || !val)) return E3_ERR_INVALID_ARG;
  for (int64_t k = 0; k < m; ++k) {
    i0[k] = p->recs[k].i0, i1[k] = p->recs[k].i1, i2[k] = p->recs[k].i2, val[k] = p->recs[k].v;
  }
  return E3_OK;
}

e3_status e3_sh_host(int lmax, const double* u, double* y, int64_t n) {
  if (lmax < 0 || lmax > 3 || n < 0 || (n > 0 && (!u || !y))) return E3_ERR_INVALID_ARG;
  e3b::ShTable t = e3b::sh_table(lmax);
  const int d = (lmax + 1) * (lmax + 1);
  for (int64_t i = 0; i < n; ++i) e3b::sh_eval(t, u + 3 * i, y + d * i);
  return E3_OK;
}

namespace {
// Both sorts of the graph build: ceil(nbits / 8) passes ping-ponging between
// (tk, ti) and the outputs, so that the last lands in (keys_out, ids_out).
struct SortBufs {
  uint32_t *keys, *keys_out, *tk;
  int32_t *ids_out, *ti, *count;  // count: 256 * (sort_tiles(n) + 1)
};
hipError_t sort_pairs(const SortBufs (&s)[2], int64_t n, int nbits, int* bad, hipStream_t st) {
  const int64_t tiles = sort_tiles(n);
  const int passes = (nbits + 7) / 8;
  SortPass a{};
  for (int k = 0; k < 2; ++k) a.kin[k] = s[k].keys, a.iin[k] = nullptr, a.count[k] = s[k].count;
  for (int p = 0; p < passes; ++p) {
    const bool to_out = ((passes - 1 - p) % 2) == 0;
    for (int k = 0; k < 2; ++k)
      a.kout[k] = to_out ? s[k].keys_out : s[k].tk, a.iout[k] = to_out ? s[k].ids_out : s[k].ti;
    const dim3 grid((unsigned)tiles, 2), block(kSortBlock);
    const bool few = n <= kSortLarge;
    hipLaunchKernelGGL(few ? k_sort_hist<4> : k_sort_hist<16>, grid, block, 0, st, a, n, 8 * p, tiles);
    hipLaunchKernelGGL(k_sort_scan, dim3(256, 2), block, 0, st, a, tiles);
    hipLaunchKernelGGL(few ? k_sort_scatter<4> : k_sort_scatter<16>, grid, block, 0, st, a, n, 8 * p, tiles, bad);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    for (int k = 0; k < 2; ++k) a.kin[k] = a.kout[k], a.iin[k] = a.iout[k];
  }
  return hipSuccess;
}
}  // namespace

e3_status e3_graph_create(const int32_t* sender, const int32_t* receiver, int64_t n_nodes, int64_t n_edges,
                          int32_t pad_node, e3_stream stream, e3_graph** out) {
  if (!out) return E3_ERR_INVALID_ARG;
  *out = nullptr;
  if (n_nodes < 0 || n_edges < 0 || n_nodes >= INT32_MAX || n_edges >= INT32_MAX) return E3_ERR_INVALID_ARG;
  if (n_edges > 0 && (!sender || !receiver)) return E3_ERR_INVALID_ARG;
  if (pad_node < -1 || (pad_node >= 0 && pad_node >= n_nodes)) return E3_ERR_INVALID_ARG;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  e3_graph* g = new (std::nothrow) e3_graph();
  if (!g) return E3_ERR_ALLOC;
  g->n_nodes = n_nodes, g->n_edges = n_edges, g->pad = pad_node;
  const int64_t E = n_edges, N = n_nodes;
  auto fail = [&](e3_status s) {
    e3_graph_destroy(g);
    return s;
  };
  // One allocation for the graph's arrays and one for the sorts' temporaries:
  // 14 of them, their frees and a second wait took most of a small graph's
  // build (1,503 atoms, 87,000 edges: build and destruction together about 205 ->
  // 105 us, with the sorts' shorter tiles and shared launches).  The arrays that
  // are written last serve the sorts first.
  const size_t nb = align256((size_t)(N + 1) * 4), eb = align256(std::max<size_t>((size_t)E * 4, 4));
  const int64_t tiles = sort_tiles(E);
  const size_t cb = align256((size_t)256 * (tiles + 1) * 4);
  char* tmp = nullptr;
  if (hipMalloc(&g->mem, 2 * nb + 5 * eb) != hipSuccess || hipMalloc((void**)&tmp, 5 * eb + 2 * cb + 256) != hipSuccess) {
    g_last_error = "hipMalloc failed in e3_graph_create";
    return fail(E3_ERR_ALLOC);  // tmp is the last to be allocated
  }
  auto take = [](char*& at, size_t bytes) {
    char* p = at;
    at += bytes;
    return reinterpret_cast<int32_t*>(p);
  };
  char* at = static_cast<char*>(g->mem);
  g->rowptr_r = take(at, nb), g->rowptr_s = take(at, nb);
  g->eid_r = take(at, eb), g->eid_s = take(at, eb), g->src_r = take(at, eb), g->r2s = take(at, eb);
  g->pos_s = take(at, eb);
  at = tmp;
  auto key = [&]() { return reinterpret_cast<uint32_t*>(take(at, eb)); };
  SortBufs sb[2];
  sb[0] = {key(), key(), reinterpret_cast<uint32_t*>(g->src_r), g->eid_r, g->r2s, nullptr};
  sb[1] = {key(), key(), key(), g->eid_s, g->pos_s, nullptr};
  sb[0].count = take(at, cb), sb[1].count = take(at, cb);
  int* flag = take(at, 256);  // index out of range, inconsistent offsets, live edges
  // keys are receivers (senders) in [0, N), padding edges N
  int end_bit = 1;
  while (end_bit < 32 && ((int64_t)1 << end_bit) <= N) ++end_bit;
  hipError_t herr = hipMemsetAsync(flag, 0, 3 * sizeof(int), st);
  if (herr == hipSuccess && E > 0) {
    hipLaunchKernelGGL(k_graph_keys, dim3(blocks_for(E, 256)), dim3(256), 0, st, sender, receiver, E, (int32_t)N,
                       pad_node, sb[0].keys, sb[1].keys, flag);
    herr = hipGetLastError();
    if (herr == hipSuccess) herr = sort_pairs(sb, E, end_bit, flag + 1, st);
    if (herr == hipSuccess) {
      hipLaunchKernelGGL(k_graph_rowptr, dim3(blocks_for(N + 1, 256), 2), dim3(256), 0, st, sb[0].keys_out,
                         sb[1].keys_out, E, (int32_t)N, g->rowptr_r, g->rowptr_s, flag + 2);
      hipLaunchKernelGGL(k_graph_finish, dim3(blocks_for(E, 256)), dim3(256), 0, st, sender, g->eid_r, g->eid_s,
                         flag, g->src_r, g->pos_s);
      hipLaunchKernelGGL(k_graph_r2s, dim3(blocks_for(E, 256)), dim3(256), 0, st, g->eid_r, g->pos_s, flag,
                         g->r2s);
      herr = hipGetLastError();
    }
  } else if (herr == hipSuccess) {
    herr = hipMemsetAsync(g->rowptr_r, 0, 2 * nb, st);
  }
  int host[3] = {0, 0, 0};
  if (herr == hipSuccess) herr = hipMemcpyAsync(host, flag, 3 * sizeof(int), hipMemcpyDeviceToHost, st);
  if (herr == hipSuccess) herr = hipStreamSynchronize(st);
  (void)hipFree(tmp);
  if (herr != hipSuccess) {
    g_last_error = std::string("e3_graph_create: ") + hipGetErrorString(herr);
    return fail(E3_ERR_HIP);
  }
  if (host[0]) return fail(E3_ERR_INDEX_OUT_OF_RANGE);
  if (host[1]) {
    g_last_error = "e3_graph_create: inconsistent sort offsets";
    return fail(E3_ERR_HIP);
  }
  g->n_live = host[2];
  g->n_pad = E - g->n_live;
  *out = g;
  return E3_OK;
}

e3_status e3_graph_live_edges(const e3_graph* g, int64_t* n_live) {
  if (!g || !n_live) return E3_ERR_INVALID_ARG;
  *n_live = g->n_live;
  return E3_OK;
}

e3_status e3_graph_export(const e3_graph* g, int32_t* perm_r, int32_t* rowptr_r, int32_t* perm_s, int32_t* rowptr_s) {
  if (!g) return E3_ERR_INVALID_ARG;
  const size_t nl = (size_t)g->n_live * 4, nr = (size_t)(g->n_nodes + 1) * 4;
  if (perm_r && nl) E3_HIP(hipMemcpy(perm_r, g->eid_r, nl, hipMemcpyDeviceToDevice));
  if (rowptr_r) E3_HIP(hipMemcpy(rowptr_r, g->rowptr_r, nr, hipMemcpyDeviceToDevice));
  if (perm_s && nl) E3_HIP(hipMemcpy(perm_s, g->eid_s, nl, hipMemcpyDeviceToDevice));
  if (rowptr_s) E3_HIP(hipMemcpy(rowptr_s, g->rowptr_s, nr, hipMemcpyDeviceToDevice));
  return E3_OK;
}

e3_status e3_graph_destroy(e3_graph* g) {
  if (!g) return E3_OK;
  (void)hipFree(g->mem);
  delete g;
  return E3_OK;
}

e3_status e3_sh(int lmax, const float* vec, float* y, int64_t n, e3_stream stream) {
  if (lmax < 0 || lmax > 3 || n < 0 || (n > 0 && (!vec || !y))) return E3_ERR_INVALID_ARG;
  if (n == 0) return E3_OK;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const dim3 grid(blocks_for(n, 256));
  TimedLaunch t_("sh", st);
  switch (lmax) {
    case 0: hipLaunchKernelGGL(k_sh<0>, grid, dim3(256), 0, st, vec, y, n); break;
    case 1: hipLaunchKernelGGL(k_sh<1>, grid, dim3(256), 0, st, vec, y, n); break;
    case 2: hipLaunchKernelGGL(k_sh<2>, grid, dim3(256), 0, st, vec, y, n); break;
    default: hipLaunchKernelGGL(k_sh<3>, grid, dim3(256), 0, st, vec, y, n); break;
  }
  E3_HIP(hipGetLastError());
  return E3_OK;
}

e3_status e3_sh_bwd(int lmax, const float* vec, const float* dy, float* dvec, int64_t n, e3_stream stream) {
  if (lmax < 0 || lmax > 3 || n < 0 || (n > 0 && (!vec || !dy || !dvec))) return E3_ERR_INVALID_ARG;
  if (n == 0) return E3_OK;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const dim3 grid(blocks_for(n, 256));
  TimedLaunch t_("sh_bwd", st);
  switch (lmax) {
    case 0: hipLaunchKernelGGL(k_sh_bwd<0>, grid, dim3(256), 0, st, vec, dy, dvec, n); break;
    case 1: hipLaunchKernelGGL(k_sh_bwd<1>, grid, dim3(256), 0, st, vec, dy, dvec, n); break;
    case 2: hipLaunchKernelGGL(k_sh_bwd<2>, grid, dim3(256), 0, st, vec, dy, dvec, n); break;
    default: hipLaunchKernelGGL(k_sh_bwd<3>, grid, dim3(256), 0, st, vec, dy, dvec, n); break;
  }
  E3_HIP(hipGetLastError());
  return E3_OK;
}

e3_status e3_tp_fwd(const e3_plan* p, const float* x, const float* y, const float* w, float* z, int64_t rows,
                    e3_stream stream) {
  e3_status s = check_any(p);
  if (s != E3_OK) return s;
  if (rows < 0) return E3_ERR_INVALID_ARG;
  if (rows > 0 && (!x || !y || !w || !z || !aligned16(x) || !aligned16(w) || !aligned16(z))) return E3_ERR_INVALID_ARG;
  if (rows == 0) return E3_OK;
  if (p->variant < 0) return rec_fwd(p, nullptr, rows, x, nullptr, y, w, z, 0, reinterpret_cast<hipStream_t>(stream));
  const VariantOps& v = (*kVariants[p->variant]());
  return v.tp[p->cpl_f == 1 ? 0 : 1](p, x, y, w, z, rows, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_tp_workspace_size(const e3_plan* p, int64_t rows, size_t* bwd_bytes) {
  e3_status s = check_any(p);
  if (s != E3_OK) return s;
  if (rows < 0 || !bwd_bytes) return E3_ERR_INVALID_ARG;
  *bwd_bytes = p->variant >= 0 ? (*kVariants[p->variant]()).tpws(p, rows) : rec_tp_ws(p, rows);
  return E3_OK;
}

e3_status e3_tp_bwd(const e3_plan* p, const float* x, const float* y, const float* w, const float* dz, float* dx,
                    float* dy, float* dw, void* ws, size_t ws_bytes, int64_t rows, e3_stream stream) {
  e3_status s = check_any(p);
  if (s != E3_OK) return s;
  if (rows < 0) return E3_ERR_INVALID_ARG;
  if (rows == 0) return E3_OK;
  if (!x || !y || !w || !dz || !dx || !dy || !dw || !ws || !aligned16(x) || !aligned16(w) || !aligned16(dz) ||
      !aligned16(dx) || !aligned16(dw) || !aligned16(ws))
    return E3_ERR_INVALID_ARG;
  if (p->variant < 0) {
    if (ws_bytes < rec_tp_ws(p, rows)) return E3_ERR_WORKSPACE_TOO_SMALL;
    return rec_bwd(p, nullptr, rows, x, nullptr, y, w, dz, dx, nullptr, dy, dw, 0, ws,
                   reinterpret_cast<hipStream_t>(stream));
  }
  const VariantOps& v = (*kVariants[p->variant]());
  if (ws_bytes < v.tpws(p, rows)) return E3_ERR_WORKSPACE_TOO_SMALL;
  return v.tpb(p, x, y, w, dz, dx, dy, dw, ws, rows, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_workspace_size(const e3_plan* p, const e3_graph* g, size_t* fwd_bytes, size_t* bwd_bytes) {
  e3_status s = check_any(p);
  if (s != E3_OK) return s;
  if (!g) return E3_ERR_INVALID_ARG;
  Ws w = conv_ws(p, g);
  if (fwd_bytes) *fwd_bytes = 0;
  if (bwd_bytes) *bwd_bytes = w.t_bytes + w.dy_bytes;
  return E3_OK;
}

e3_status e3_conv_fwd(const e3_plan* p, const e3_graph* g, const float* x, const float* vec, const float* s,
                      float* m, void* ws, size_t ws_bytes, e3_stream stream) {
  (void)ws, (void)ws_bytes;
  e3_status st = check_any(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!m || !aligned16(m) || !x || !aligned16(x))) return E3_ERR_INVALID_ARG;
  if (g->n_live > 0 && (!vec || !s || !aligned16(s))) return E3_ERR_INVALID_ARG;
  if (p->variant < 0) return rec_fwd(p, g, 0, x, vec, nullptr, s, m, 0, reinterpret_cast<hipStream_t>(stream));
  const VariantOps& v = (*kVariants[p->variant]());
  return v.fwd(p, g, x, vec, nullptr, s, m, 0, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_bwd(const e3_plan* p, const e3_graph* g, const float* x, const float* vec, const float* s,
                      const float* dm, float* dx, float* dvec, float* ds, void* ws, size_t ws_bytes,
                      e3_stream stream) {
  e3_status st = check_any(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !dm || !dx || !aligned16(x) || !aligned16(dm) || !aligned16(dx)))
    return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!vec || !s || !ds || !dvec || !aligned16(s) || !aligned16(ds))) return E3_ERR_INVALID_ARG;
  Ws w = conv_ws(p, g);
  if (w.t_bytes + w.dy_bytes > 0 && (!ws || !aligned16(ws))) return E3_ERR_INVALID_ARG;
  if (ws_bytes < w.t_bytes + w.dy_bytes) return E3_ERR_WORKSPACE_TOO_SMALL;
  if (p->variant < 0)
    return rec_bwd(p, g, 0, x, vec, nullptr, s, dm, dx, dvec, nullptr, ds, 0, ws,
                   reinterpret_cast<hipStream_t>(stream));
  const VariantOps& v = (*kVariants[p->variant]());
  return v.bwd(p, g, x, vec, nullptr, s, dm, dx, dvec, nullptr, ds, 0, ws, reinterpret_cast<hipStream_t>(stream));
}

// ---- float64 builds
e3_status e3_tp_fwd_f64(const e3_plan* p, const double* x, const double* y, const double* w, double* z,
                        int64_t rows, e3_stream stream) {
  e3_status s = check_composable(p);
  if (s != E3_OK) return s;
  if (rows < 0) return E3_ERR_INVALID_ARG;
  if (rows == 0) return E3_OK;
  if (!x || !y || !w || !z || !aligned16(x) || !aligned16(w) || !aligned16(z)) return E3_ERR_INVALID_ARG;
  if (p->variant < 0) return comp_tp64(p, x, y, w, z, rows, reinterpret_cast<hipStream_t>(stream));
  return (*kVariants[p->variant]()).tp64(p, x, y, w, z, rows, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_tp_workspace_size_f64(const e3_plan* p, int64_t rows, size_t* bwd_bytes) {
  e3_status s = check_composable(p);
  if (s != E3_OK) return s;
  if (rows < 0 || !bwd_bytes) return E3_ERR_INVALID_ARG;
  *bwd_bytes = p->variant >= 0 ? (*kVariants[p->variant]()).tpws64(p, rows) : comp_tp_ws64(p, rows);
  return E3_OK;
}

e3_status e3_tp_bwd_f64(const e3_plan* p, const double* x, const double* y, const double* w, const double* dz,
                        double* dx, double* dy, double* dw, void* ws, size_t ws_bytes, int64_t rows,
                        e3_stream stream) {
  e3_status s = check_composable(p);
  if (s != E3_OK) return s;
  if (rows < 0) return E3_ERR_INVALID_ARG;
  if (rows == 0) return E3_OK;
  if (!x || !y || !w || !dz || !dx || !dy || !dw || !ws || !aligned16(x) || !aligned16(w) || !aligned16(dz) ||
      !aligned16(dx) || !aligned16(dw) || !aligned16(ws))
    return E3_ERR_INVALID_ARG;
  if (p->variant < 0) {
    if (ws_bytes < comp_tp_ws64(p, rows)) return E3_ERR_WORKSPACE_TOO_SMALL;
    return comp_tpb64(p, x, y, w, dz, dx, dy, dw, ws, rows, reinterpret_cast<hipStream_t>(stream));
  }
  const VariantOps& v = (*kVariants[p->variant]());
  if (ws_bytes < v.tpws64(p, rows)) return E3_ERR_WORKSPACE_TOO_SMALL;
  return v.tpb64(p, x, y, w, dz, dx, dy, dw, ws, rows, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_workspace_size_f64(const e3_plan* p, const e3_graph* g, size_t* bwd_bytes) {
  e3_status s = check_composable(p);
  if (s != E3_OK) return s;
  if (!g || !bwd_bytes) return E3_ERR_INVALID_ARG;
  const Ws w = p->variant >= 0 ? (*kVariants[p->variant]()).ws64(p, g) : comp_ws64(p, g);
  *bwd_bytes = w.t_bytes + w.dy_bytes;
  return E3_OK;
}

e3_status e3_conv_fwd_f64(const e3_plan* p, const e3_graph* g, const double* x, const double* vec, const double* s,
                          double* m, e3_stream stream) {
  e3_status st = check_composable(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !m || !aligned16(x) || !aligned16(m))) return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!vec || !s || !aligned16(s))) return E3_ERR_INVALID_ARG;
  if (p->variant < 0) return comp_fwd64(p, g, x, vec, s, m, reinterpret_cast<hipStream_t>(stream));
  return (*kVariants[p->variant]()).fwd64(p, g, x, vec, s, m, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_bwd_f64(const e3_plan* p, const e3_graph* g, const double* x, const double* vec, const double* s,
                          const double* dm, double* dx, double* dvec, double* ds, void* ws, size_t ws_bytes,
                          e3_stream stream) {
  e3_status st = check_composable(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !dm || !dx || !aligned16(x) || !aligned16(dm) || !aligned16(dx)))
    return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!vec || !s || !ds || !dvec || !aligned16(s) || !aligned16(ds))) return E3_ERR_INVALID_ARG;
  const Ws w = p->variant >= 0 ? (*kVariants[p->variant]()).ws64(p, g) : comp_ws64(p, g);
  if (w.t_bytes + w.dy_bytes > 0 && (!ws || !aligned16(ws))) return E3_ERR_INVALID_ARG;
  if (ws_bytes < w.t_bytes + w.dy_bytes) return E3_ERR_WORKSPACE_TOO_SMALL;
  if (p->variant < 0)
    return comp_bwd64(p, g, x, vec, s, dm, dx, dvec, ds, ws, reinterpret_cast<hipStream_t>(stream));
  return (*kVariants[p->variant]()).bwd64(p, g, x, vec, s, dm, dx, dvec, ds, ws,
                                          reinterpret_cast<hipStream_t>(stream));
}

}  // extern "C"

// ------------------------------------------------------------ no-allocation backward
// Scratch of e3_conv_bwd_noalloc: the per-edge x-cotangent partials and the
// per-wave harmonic-cotangent partials of the backward sweep, in a fixed
// array instead of a caller workspace.  Each device holds its own copy for the
// life of the process.  Host code never uses the array's name as an address:
// the device address comes from hipGetSymbolAddress, once per device.
constexpr size_t kNoAllocScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of `scratch`, looked up on the first call made
// with that device current.
e3_status scratch_of_current_device(void** out) {
  int dev = -1;
  E3_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    g_last_error = "device ordinal beyond the no-allocation scratch table";
    return E3_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    E3_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) {
      g_last_error = "hipGetSymbolAddress returned no address for the scratch array";
      return E3_ERR_HIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return E3_OK;
}
}  // namespace

extern "C" {

e3_status e3_conv_bwd_noalloc(const e3_plan* p, const e3_graph* g, const float* x, const float* vec,
                              const float* s, const float* dm, float* dx, float* dvec, float* ds, e3_stream stream) {
  e3_status st = check_any(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !dm || !dx || !aligned16(x) || !aligned16(dm) || !aligned16(dx)))
    return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!vec || !s || !ds || !dvec || !aligned16(s) || !aligned16(ds))) return E3_ERR_INVALID_ARG;
  const Ws w = conv_ws(p, g);
  if (w.t_bytes + w.dy_bytes > kNoAllocScratchBytes) {
    g_last_error = "the backward needs " + std::to_string(w.t_bytes + w.dy_bytes) +
                   " bytes of scratch; the no-allocation entry point has " + std::to_string(kNoAllocScratchBytes);
    return E3_ERR_WORKSPACE_TOO_SMALL;
  }
  void* ptr = nullptr;
  if ((st = scratch_of_current_device(&ptr)) != E3_OK) return st;
  // every scratch byte the kernels read is written earlier in the same call
  // (each live edge's partial rows and each wave's harmonic partials), so the
  // previous call's contents need no clearing
  if (p->variant < 0)
    return rec_bwd(p, g, 0, x, vec, nullptr, s, dm, dx, dvec, nullptr, ds, 0, ptr,
                   reinterpret_cast<hipStream_t>(stream));
  const VariantOps& v = (*kVariants[p->variant]());
  return v.bwd(p, g, x, vec, nullptr, s, dm, dx, dvec, nullptr, ds, 0, ptr, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_radial_workspace_size(const e3_plan* p, const e3_graph* g, int K, size_t* bwd_bytes) {
  e3_status st = check_composable(p);
  if (st != E3_OK) return st;
  if (!g || !bwd_bytes || K < 1 || K > kRadKMax) return E3_ERR_INVALID_ARG;
  *bwd_bytes = p->variant >= 0 ? (*kVariants[p->variant]()).rws(p, g, K).total() : comp_rad_ws(p, g, K).total();
  return E3_OK;
}

e3_status e3_conv_fwd_radial(const e3_plan* p, const e3_graph* g, const float* x, const float* vec, const float* h,
                             const float* W, int K, float* m, e3_stream stream) {
  e3_status st = check_composable(p);
  if (st != E3_OK) return st;
  if (!g || K < 1 || K > kRadKMax) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!m || !aligned16(m) || !x || !aligned16(x) || !W || !aligned16(W))) return E3_ERR_INVALID_ARG;
  if (g->n_live > 0 && (!vec || !h)) return E3_ERR_INVALID_ARG;
  if (p->variant < 0) return comp_fwd_rad(p, g, x, vec, h, W, K, m, reinterpret_cast<hipStream_t>(stream));
  return (*kVariants[p->variant]()).rfwd(p, g, x, vec, h, W, K, m, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_bwd_radial(const e3_plan* p, const e3_graph* g, const float* x, const float* vec, const float* h,
                             const float* W, int K, const float* dm, float* dx, float* dvec, float* dh, float* dW,
                             void* ws, size_t ws_bytes, e3_stream stream) {
  e3_status st = check_composable(p);
  if (st != E3_OK) return st;
  if (!g || K < 1 || K > kRadKMax || !W || !aligned16(W) || !dW) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !dm || !dx || !aligned16(x) || !aligned16(dm) || !aligned16(dx)))
    return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!vec || !h || !dh || !dvec)) return E3_ERR_INVALID_ARG;
  const RadWs w = p->variant >= 0 ? (*kVariants[p->variant]()).rws(p, g, K) : comp_rad_ws(p, g, K);
  if (w.total() > 0 && (!ws || !aligned16(ws))) return E3_ERR_INVALID_ARG;
  if (ws_bytes < w.total()) return E3_ERR_WORKSPACE_TOO_SMALL;
  if (p->variant < 0)
    return comp_bwd_rad(p, g, x, vec, h, W, K, dm, dx, dvec, dh, dW, ws, reinterpret_cast<hipStream_t>(stream));
  return (*kVariants[p->variant]()).rbwd(p, g, x, vec, h, W, K, dm, dx, dvec, dh, dW, ws,
                                         reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_fwd_y(const e3_plan* p, const e3_graph* g, const float* x, const float* y, const float* s,
                        float* m, int accumulate, e3_stream stream) {
  e3_status st = check_any(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!m || !aligned16(m) || !x || !aligned16(x))) return E3_ERR_INVALID_ARG;
  if (g->n_live > 0 && (!y || !s || !aligned16(s))) return E3_ERR_INVALID_ARG;
  if (p->variant < 0)
    return rec_fwd(p, g, 0, x, nullptr, y, s, m, accumulate != 0, reinterpret_cast<hipStream_t>(stream));
  const VariantOps& v = (*kVariants[p->variant]());
  return v.fwd(p, g, x, nullptr, y, s, m, accumulate != 0, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_bwd_y(const e3_plan* p, const e3_graph* g, const float* x, const float* y, const float* s,
                        const float* dm, float* dx, float* dy, float* ds, int accumulate, void* ws, size_t ws_bytes,
                        e3_stream stream) {
  e3_status st = check_any(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !dm || !aligned16(x) || !aligned16(dm) || (dx && !aligned16(dx))))
    return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!y || !s || !aligned16(s) || (ds && !aligned16(ds)))) return E3_ERR_INVALID_ARG;
  Ws w = conv_ws(p, g);
  if (w.t_bytes + w.dy_bytes > 0 && (!ws || !aligned16(ws))) return E3_ERR_INVALID_ARG;
  if (ws_bytes < w.t_bytes + w.dy_bytes) return E3_ERR_WORKSPACE_TOO_SMALL;
  if (p->variant < 0)
    return rec_bwd(p, g, 0, x, nullptr, y, s, dm, dx, nullptr, dy, ds, accumulate ? (kAccDx | kAccDy | kAccDs) : 0,
                   ws, reinterpret_cast<hipStream_t>(stream));
  const VariantOps& v = (*kVariants[p->variant]());
  return v.bwd(p, g, x, nullptr, y, s, dm, dx, nullptr, dy, ds, accumulate ? (kAccDx | kAccDy | kAccDs) : 0, ws,
               reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_conv_bwd2(const e3_plan* p, const e3_graph* g, const float* x, const float* y, const float* s,
                       const float* dm, const float* ddx, const float* ddy, const float* dds, float* gx, float* gy,
                       float* gs, float* gdm, void* ws, size_t ws_bytes, e3_stream stream) {
  e3_status st = check_any(p);
  if (st != E3_OK) return st;
  if (!g) return E3_ERR_INVALID_ARG;
  if (g->n_nodes > 0 && (!x || !dm || !ddx || !gx || !gdm || !aligned16(x) || !aligned16(dm) || !aligned16(ddx) ||
                         !aligned16(gx) || !aligned16(gdm)))
    return E3_ERR_INVALID_ARG;
  if (g->n_edges > 0 && (!y || !s || !ddy || !dds || !gy || !gs || !aligned16(s) || !aligned16(dds) ||
                         !aligned16(gs)))
    return E3_ERR_INVALID_ARG;
  Ws w = conv_ws(p, g);
  if (w.t_bytes + w.dy_bytes > 0 && (!ws || !aligned16(ws))) return E3_ERR_INVALID_ARG;
  if (ws_bytes < w.t_bytes + w.dy_bytes) return E3_ERR_WORKSPACE_TOO_SMALL;
  hipStream_t hs = reinterpret_cast<hipStream_t>(stream);
  if (p->composed) return comp_bwd2(p, g, x, y, s, dm, ddx, ddy, dds, gx, gy, gs, gdm, ws, hs);
  if (p->variant < 0) {  // the record path: three forward and three backward calls
    if ((st = rec_fwd(p, g, 0, ddx, nullptr, y, s, gdm, 0, hs)) != E3_OK) return st;
    if ((st = rec_fwd(p, g, 0, x, nullptr, ddy, s, gdm, 1, hs)) != E3_OK) return st;
    if ((st = rec_fwd(p, g, 0, x, nullptr, y, dds, gdm, 1, hs)) != E3_OK) return st;
    if ((st = rec_bwd(p, g, 0, ddx, nullptr, y, s, dm, nullptr, nullptr, gy, gs, 0, ws, hs)) != E3_OK) return st;
    if ((st = rec_bwd(p, g, 0, x, nullptr, ddy, s, dm, gx, nullptr, nullptr, gs, kAccDs, ws, hs)) != E3_OK)
      return st;
    return rec_bwd(p, g, 0, x, nullptr, y, dds, dm, gx, nullptr, gy, nullptr, kAccDx | kAccDy, ws, hs);
  }
  const VariantOps& v = (*kVariants[p->variant]());
  // ddm = conv(ddx, y, s) + conv(x, ddy, s) + conv(x, y, dds), in one pass
  if ((st = v.fwd3(p, g, x, ddx, y, ddy, s, dds, gdm, hs)) != E3_OK) return st;
  // gx, gy, gs in one sweep
  return v.bwd3(p, g, x, ddx, y, ddy, s, dds, dm, gx, gy, gs, ws, hs);
}

}  // extern "C"

// ============================================================ linear mixing (host)
struct e3_linear {
  int d_in = 0, d_out = 0, c_in = 0, c_out = 0;
  int64_t nw = 0;
  std::vector<LinJob> fj, bj;   // forward jobs (output blocks), dx jobs (input blocks)
  std::vector<LinSrc> fs, bs;
  std::vector<LinPair> pairs;
  char* dev = nullptr;  // device copy of the tables (uploaded by e3_linear_create)
  int device = -1;      // the device that holds it
  size_t off_fj = 0, off_fs = 0, off_bj = 0, off_bs = 0, off_pairs = 0;
};

namespace {
// Device copy of the job and pair tables, on the current device (synchronous:
// called once, from e3_linear_create).
e3_status lin_upload(e3_linear* L) {
  size_t off = 0;
  auto place = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
  L->off_fj = place(L->fj.size() * sizeof(LinJob) + 1);
  L->off_fs = place(L->fs.size() * sizeof(LinSrc) + 1);
  L->off_bj = place(L->bj.size() * sizeof(LinJob) + 1);
  L->off_bs = place(L->bs.size() * sizeof(LinSrc) + 1);
  L->off_pairs = place(L->pairs.size() * sizeof(LinPair) + 1);
  std::vector<char> host(off, 0);
  auto put = [&](size_t o, const void* p, size_t b) { if (b) std::memcpy(host.data() + o, p, b); };
  put(L->off_fj, L->fj.data(), L->fj.size() * sizeof(LinJob));
  put(L->off_fs, L->fs.data(), L->fs.size() * sizeof(LinSrc));
  put(L->off_bj, L->bj.data(), L->bj.size() * sizeof(LinJob));
  put(L->off_bs, L->bs.data(), L->bs.size() * sizeof(LinSrc));
  put(L->off_pairs, L->pairs.data(), L->pairs.size() * sizeof(LinPair));
  E3_HIP(hipGetDevice(&L->device));
  char* d = nullptr;
  E3_HIP(hipMalloc(&d, off));
  const hipError_t e = hipMemcpy(d, host.data(), off, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    g_last_error = std::string("linear tables upload: ") + hipGetErrorString(e);
    (void)hipFree(d);
    return E3_ERR_HIP;
  }
  L->dev = d;
  return E3_OK;
}

// The tables live on the device current at creation; a call made with another
// device current is refused rather than reading another device's memory.
e3_status check_device(int device, const char* what) {
  int cur = -1;
  E3_HIP(hipGetDevice(&cur));
  if (cur != device) {
    g_last_error = std::string(what) + " was created on device " + std::to_string(device) +
                   ", called with device " + std::to_string(cur) + " current";
    return E3_ERR_INVALID_ARG;
  }
  return E3_OK;
}

// Tile width of an operand of C columns: the one of 64 and 128 with fewer padded ones.
int lin_tile(int C) { return (C + 63) / 64 % 2 ? 64 : 128; }
constexpr int kLinRows = 128;  // rows of a gather-GEMM tile

// wt: W is read transposed ([col][k], 16-byte aligned).
e3_status lin_gemm(const std::vector<LinJob>& jobs, const LinJob* djobs, const LinSrc* dsrcs, const float* src,
                   const float* W, bool wt, float* dst, int64_t n, int D_src, int C_src, int D_dst, int C_dst,
                   const char* name, hipStream_t st) {
  const int bn = lin_tile(C_dst);
  LinArgs a{};
  a.src = src, a.W = W, a.dst = dst, a.jobs = djobs, a.srcs = dsrcs, a.n = n;
  a.D_src = D_src, a.C_src = C_src, a.D_dst = D_dst, a.C_dst = C_dst;
  a.njobs = (int)jobs.size();
  a.slabs = (C_dst + bn - 1) / bn;
  int64_t u = 0;
  for (size_t j = 0; j < jobs.size(); ++j) {
    a.first[j] = (int)u;
    u += (n * jobs[j].R + kLinRows - 1) / kLinRows * a.slabs;
  }
  a.first[jobs.size()] = (int)u;
  if (u == 0) return E3_OK;
  if (u > 0x7fffffff) return E3_ERR_INVALID_ARG;
  auto* k = wt ? (bn == 128 ? k_lin_gemm<kLinRows, 128, true> : k_lin_gemm<kLinRows, 64, true>)
               : (bn == 128 ? k_lin_gemm<kLinRows, 128, false> : k_lin_gemm<kLinRows, 64, false>);
  TimedLaunch t_(name, st);
  hipLaunchKernelGGL(k, grid_of(u), dim3(kSpThreads), 0, st, a);
  E3_HIP(hipGetLastError());
  return E3_OK;
}

// dW partials, then W transposed slice by slice (read by dx along rows)
size_t lin_ws_dwp(const e3_linear* L) {
  return align256((size_t)L->pairs.size() * kLinChunks * L->c_in * L->c_out * sizeof(float));
}
size_t lin_ws(const e3_linear* L) { return lin_ws_dwp(L) + align256((size_t)L->nw * sizeof(float)); }
}  // namespace

extern "C" {

e3_status e3_linear_create(const char* irreps_in, const char* irreps_out, e3_linear** out) {
  if (!irreps_in || !irreps_out || !out) return E3_ERR_INVALID_ARG;
  *out = nullptr;
  std::vector<e3b::Block> bi, bo;
  std::string err;
  if (!e3b::parse_irreps(irreps_in, bi, err) || !e3b::parse_irreps(irreps_out, bo, err)) {
    g_last_error = err;
    return E3_ERR_INVALID_ARG;
  }
  const int c_in = bi[0].mul, c_out = bo[0].mul;
  for (const auto& b : bi)
    if (b.mul != c_in) return E3_ERR_INVALID_ARG;
  for (const auto& b : bo)
    if (b.mul != c_out) return E3_ERR_INVALID_ARG;
  if (c_in % 16 || c_out % 16 || c_in > 4096 || c_out > 4096) {
    g_last_error = "linear mixing needs multiplicities that are multiples of 16 (at most 4096)";
    return E3_ERR_UNSUPPORTED;
  }
  if ((int)bi.size() > kLinMaxJobs || (int)bo.size() > kLinMaxJobs) {
    g_last_error = "linear mixing supports at most 64 blocks per side";
    return E3_ERR_UNSUPPORTED;
  }
  e3_linear* L = new (std::nothrow) e3_linear();
  if (!L) return E3_ERR_ALLOC;
  L->c_in = c_in, L->c_out = c_out;
  std::vector<int> irow(bi.size()), orow(bo.size());
  for (size_t i = 0; i < bi.size(); ++i) irow[i] = L->d_in, L->d_in += 2 * bi[i].l + 1;
  for (size_t o = 0; o < bo.size(); ++o) orow[o] = L->d_out, L->d_out += 2 * bo[o].l + 1;
  // forward: one job per output block, sources = input blocks of its type, in order
  std::vector<std::vector<std::pair<int, int64_t>>> feeds(bi.size());  // input -> (output, W offset)
  int64_t woff = 0;
  for (size_t o = 0; o < bo.size(); ++o) {
    LinJob j{2 * bo[o].l + 1, orow[o], (int)L->fs.size(), 0};
    for (size_t i = 0; i < bi.size(); ++i)
      if (bi[i].l == bo[o].l && bi[i].p == bo[o].p) {
        L->fs.push_back(LinSrc{irow[i], 0, woff});
        L->pairs.push_back(LinPair{j.R, irow[i], orow[o], 0, woff});
        feeds[i].push_back({(int)o, woff});
        woff += (int64_t)c_in * c_out;
        ++j.nsrc;
      }
    L->fj.push_back(j);
  }
  L->nw = woff;
  // dx: one job per input block, sources = the output blocks it feeds (W read transposed)
  for (size_t i = 0; i < bi.size(); ++i) {
    LinJob j{2 * bi[i].l + 1, irow[i], (int)L->bs.size(), (int)feeds[i].size()};
    for (auto& f : feeds[i]) L->bs.push_back(LinSrc{orow[f.first], 0, f.second});
    L->bj.push_back(j);
  }
  const e3_status st = lin_upload(L);
  if (st != E3_OK) {
    delete L;
    return st;
  }
  *out = L;
  return E3_OK;
}

e3_status e3_linear_query(const e3_linear* L, int64_t* n_weights, int* d_in, int* d_out, int* c_in, int* c_out) {
  if (!L) return E3_ERR_INVALID_ARG;
  if (n_weights) *n_weights = L->nw;
  if (d_in) *d_in = L->d_in;
  if (d_out) *d_out = L->d_out;
  if (c_in) *c_in = L->c_in;
  if (c_out) *c_out = L->c_out;
  return E3_OK;
}

e3_status e3_linear_destroy(e3_linear* L) {
  if (!L) return E3_OK;
  if (L->dev) (void)hipFree(L->dev);
  delete L;
  return E3_OK;
}

e3_status e3_linear_fwd(e3_linear* L, const float* x, const float* W, float* out, int64_t n, e3_stream stream) {
  if (!L || n < 0) return E3_ERR_INVALID_ARG;
  if (n == 0) return E3_OK;
  if (!x || !W || !out || !aligned16(x) || !aligned16(out)) return E3_ERR_INVALID_ARG;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  e3_status s = check_device(L->device, "linear mixing handle");
  if (s != E3_OK) return s;
  return lin_gemm(L->fj, reinterpret_cast<const LinJob*>(L->dev + L->off_fj),
                  reinterpret_cast<const LinSrc*>(L->dev + L->off_fs), x, W, false, out, n, L->d_in, L->c_in,
                  L->d_out, L->c_out, "linear_fwd", st);
}

e3_status e3_linear_workspace_size(const e3_linear* L, size_t* bwd_bytes) {
  if (!L || !bwd_bytes) return E3_ERR_INVALID_ARG;
  *bwd_bytes = lin_ws(L);
  return E3_OK;
}

e3_status e3_linear_bwd(e3_linear* L, const float* x, const float* W, const float* dout, float* dx, float* dW,
                        void* ws, size_t ws_bytes, int64_t n, e3_stream stream) {
  if (!L || n < 0) return E3_ERR_INVALID_ARG;
  if (!W || !dW || (n > 0 && (!x || !dout || !dx || !aligned16(x) || !aligned16(dout) || !aligned16(dx))))
    return E3_ERR_INVALID_ARG;
  if (ws_bytes < lin_ws(L)) return E3_ERR_WORKSPACE_TOO_SMALL;
  if (lin_ws(L) > 0 && (!ws || !aligned16(ws))) return E3_ERR_INVALID_ARG;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  e3_status s = check_device(L->device, "linear mixing handle");
  if (s != E3_OK) return s;
  const LinPair* dp = reinterpret_cast<const LinPair*>(L->dev + L->off_pairs);
  if (n > 0) {
    // slices of Wt sit at the same offsets as those of W (pair order)
    float* Wt = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + lin_ws_dwp(L));
    const bool wt = aligned16(W);
    if (!L->pairs.empty() && !wt) {
      TimedLaunch t_("linear_bwd_transpose", st);
      hipLaunchKernelGGL(k_lin_transpose, dim3(blocks_for(L->nw, 256)), dim3(256), 0, st, W, dp, Wt,
                         (int)L->pairs.size(), L->c_in, L->c_out);
      E3_HIP(hipGetLastError());
    }
    s = lin_gemm(L->bj, reinterpret_cast<const LinJob*>(L->dev + L->off_bj),
                 reinterpret_cast<const LinSrc*>(L->dev + L->off_bs), dout, wt ? W : Wt, wt, dx, n, L->d_out,
                 L->c_out, L->d_in, L->c_in, "linear_bwd_dx", st);
    if (s != E3_OK) return s;
  }
  if (L->pairs.empty()) return E3_OK;
  float* dWp = reinterpret_cast<float*>(ws);
  LinDwArgs a{};
  a.x = x, a.dout = dout, a.dWp = dWp, a.pairs = dp, a.n = n;
  a.D_in = L->d_in, a.C_in = L->c_in, a.D_out = L->d_out, a.C_out = L->c_out;
  const int km = lin_tile(L->c_in), jm = lin_tile(L->c_out);
  a.ktiles = (L->c_in + km - 1) / km, a.jtiles = (L->c_out + jm - 1) / jm, a.npairs = (int)L->pairs.size();
  {
    auto* k = km == 128 ? (jm == 128 ? k_lin_dw<128, 128> : k_lin_dw<128, 64>)
                        : (jm == 128 ? k_lin_dw<64, 128> : k_lin_dw<64, 64>);
    TimedLaunch t_("linear_bwd_dw", st);
    const int64_t units = (int64_t)L->pairs.size() * kLinChunks * a.ktiles * a.jtiles;
    hipLaunchKernelGGL(k, grid_of(units), dim3(kSpThreads), 0, st, a);
    E3_HIP(hipGetLastError());
  }
  {
    TimedLaunch t_("linear_bwd_dw_sum", st);
    const int64_t per = (int64_t)L->c_in * L->c_out;
    hipLaunchKernelGGL(k_lin_dw_sum, dim3(blocks_for(per * (int64_t)L->pairs.size(), 256)), dim3(256), 0, st, dWp, dp,
                       dW, (int)L->pairs.size(), per);
    E3_HIP(hipGetLastError());
  }
  return E3_OK;
}

}  // extern "C"

// ============================================================ generic records (host)
struct e3_tpg {
  int d_x = 0, d_y = 0, d_z = 0, ypc = 0;
  // record tables: forward (out z, A x, B y), dx (out x, A dz, B y), dy (out y, A x, B dz)
  struct Table {
    int d_out = 0;
    std::vector<TpgRec> recs;
    std::vector<TpgRec64> recs64;
    size_t off_recs = 0, off_recs64 = 0;
  } t[3];
  char* dev = nullptr;  // device copy of the tables (uploaded by e3_tpg_create)
  int device = -1;      // the device that holds it
};

namespace {
e3_tpg::Table tpg_table(int d_out, const std::vector<std::array<int, 3>>& key, const std::vector<double>& val) {
  // key = (out, a, b); stable order by (out, a, b)
  std::vector<size_t> ord(key.size());
  for (size_t i = 0; i < ord.size(); ++i) ord[i] = i;
  std::stable_sort(ord.begin(), ord.end(), [&](size_t u, size_t v) { return key[u] < key[v]; });
  e3_tpg::Table T;
  T.d_out = d_out;
  auto push = [&](unsigned ab, double v) {
    T.recs.push_back(TpgRec{ab, (float)v});
    T.recs64.push_back(TpgRec64{ab, 0, v});
  };
  size_t k = 0;
  for (int o = 0; o < d_out; ++o) {
    if (k == ord.size() || key[ord[k]][0] != o) push(kTpgEmpty, 0.0);
    for (; k < ord.size() && key[ord[k]][0] == o; ++k) {
      const size_t i = ord[k];
      const bool last = k + 1 == ord.size() || key[ord[k + 1]][0] != o;
      push((unsigned)key[i][1] | (unsigned)key[i][2] << 10 | (last ? kTpgEnd : 0u), val[i]);
    }
  }
  while (T.recs.size() % kTpgAhead) push(0, 0.0);
  return T;
}

// Device copy of the record tables, on the current device (synchronous:
// called once, from e3_tpg_create).
e3_status tpg_upload(e3_tpg* G) {
  size_t off = 0;
  for (auto& T : G->t) {
    T.off_recs = off;
    off = align256(off + T.recs.size() * sizeof(TpgRec) + 1);
    T.off_recs64 = off;
    off = align256(off + T.recs64.size() * sizeof(TpgRec64) + 1);
  }
  std::vector<char> host(off, 0);
  for (auto& T : G->t) {
    if (!T.recs.empty()) std::memcpy(host.data() + T.off_recs, T.recs.data(), T.recs.size() * sizeof(TpgRec));
    if (!T.recs64.empty())
      std::memcpy(host.data() + T.off_recs64, T.recs64.data(), T.recs64.size() * sizeof(TpgRec64));
  }
  E3_HIP(hipGetDevice(&G->device));
  char* d = nullptr;
  E3_HIP(hipMalloc(&d, off));
  const hipError_t e = hipMemcpy(d, host.data(), off, hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    g_last_error = std::string("record tables upload: ") + hipGetErrorString(e);
    (void)hipFree(d);
    return E3_ERR_HIP;
  }
  G->dev = d;
  return E3_OK;
}

// Staging of one wave with rb pairs per lane.
size_t tpg_lds(int dA, int dB, int dout, TpgB mode, bool red, int C, size_t elem, int rb) {
  const size_t b = mode == kTpgBOwn   ? (size_t)dB * kWave * rb
                   : mode == kTpgBRow ? (size_t)(dB | 1) * tpg_tile_rows(C, rb * kWave)
                                      : (size_t)dB * rb;
  return (((size_t)dA + (red ? dout : 0)) * kWave * rb + b) * elem;
}
constexpr size_t kTpgMaxLds = 64 * 1024;
// Pairs per lane: the most of 4, 2, 1 whose staging leaves ten waves per CU,
// eight with a shared B.  More waves hide more latency, more pairs share a
// record's overhead: 118, 121 and 139 us with 2, 4 and 1 at 18 operand rows
// (30,011 rows, C = 100), 241, 292 and 281 us at 32 (20,000 rows, C = 64); a
// shared B at 16 + 16 operand rows (20,000 rows, C = 64) 155 us with 4, 207 with 2.
constexpr size_t kTpgWant = 16 * 1024, kTpgWantShared = 20 * 1024;
// Four pairs read four records ahead instead of eight where the staging leaves
// room for the waves that the registers then allow (9 + 9 rows, shared B, C =
// 128: 137 against 147 us; 16 + 16: 174 against 155), and always in float64,
// where eight take 256 registers (4 + 4 rows: 31 against 40 us).
constexpr size_t kTpgAhead4Lds = 12 * 1024;
constexpr int64_t kTpgTiles = 1024;

// What a call accepts: one row's operands of 64 channels (a shared B once)
// within the limit, and its operand block of up to four rows within 2 GiB.
size_t tpg_row_lds(int dA, int dB, int dout, bool bsh, bool red, size_t elem, int rb = 1) {
  return ((size_t)dA * rb * kWave + (bsh ? (((size_t)dB * rb + 3) & ~3) : (size_t)dB * rb * kWave) +
          (red ? (size_t)dout * rb * kWave : 0)) *
         elem;
}

template <class T>
e3_status tpg_run(const e3_tpg* G, int which, const T* A, int dA, const T* B, int dB, bool bsh, T* out, T* part,
                  bool red, int64_t rows, int C, const char* name, hipStream_t st) {
  const e3_tpg::Table& Tb = G->t[which];
  TpgArgs<T> a{};
  a.A = A, a.B = B, a.out = out, a.part = part;
  a.recs = reinterpret_cast<decltype(a.recs)>(G->dev + (sizeof(T) == 8 ? Tb.off_recs64 : Tb.off_recs));
  a.nrec = (int)Tb.recs.size();
  a.rows = rows, a.C = C, a.dA = dA, a.dB = dB;
  a.dout = Tb.d_out;
  int rows_per = 4;
  while (rows_per > 1 && tpg_row_lds(dA, dB, a.dout, bsh, red, sizeof(T), rows_per) > kTpgMaxLds) rows_per /= 2;
  if (tpg_row_lds(dA, dB, a.dout, bsh, red, sizeof(T), rows_per) > kTpgMaxLds) return E3_ERR_UNSUPPORTED;
  if ((int64_t)rows_per * std::max(dA, dB) * C * (int64_t)sizeof(T) > 0x7fffffff) return E3_ERR_INVALID_ARG;
  const TpgB mode = !bsh ? kTpgBOwn : C % kWave == 0 ? kTpgBOnce : kTpgBRow;
  int rb = 4;
  while (rb > 1 && tpg_lds(dA, dB, a.dout, mode, red, C, sizeof(T), rb) > (bsh ? kTpgWantShared : kTpgWant)) rb /= 2;
  // fewer where the tiles would not give every SIMD a wave (300 rows, C = 128, 9 +
  // 9 rows: 16 -> 13 us; 5,000 rows, C = 36, 9 + 16 rows: 45 -> 35 us)
  while (!red && rb > 1 && rows * C < (int64_t)rb * kWave * kTpgTiles) rb /= 2;
  const size_t lds = tpg_lds(dA, dB, a.dout, mode, red, C, sizeof(T), rb);
  const int pairs = rb * kWave;
  a.pieces = red ? (C + pairs - 1) / pairs : 1;
  a.rpt = red && C <= pairs ? pairs / C : 1;
  const int64_t grid = !red ? (rows * C + pairs - 1) / pairs : a.pieces > 1 ? rows * a.pieces : (rows + a.rpt - 1) / a.rpt;
  if (grid > 0x7fffffff) return E3_ERR_INVALID_ARG;
  if (red && a.pieces == 1) a.part = out;
  TimedLaunch t_(name, st);
  auto go = [&](auto RBc, auto AHc) {
    constexpr int R = decltype(RBc)::value, A = decltype(AHc)::value;
    // only a shared y's cotangent is summed, and its operands have channels
    auto* k = red                 ? k_tpg<T, kTpgBOwn, true, R, A>
              : mode == kTpgBOwn  ? k_tpg<T, kTpgBOwn, false, R, A>
              : mode == kTpgBOnce ? k_tpg<T, kTpgBOnce, false, R, A>
                                  : k_tpg<T, kTpgBRow, false, R, A>;
    // over 64 KiB only in float64 with a shared B of many rows and few channels
    if (lds > kTpgMaxLds)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k, grid_of(grid), dim3(kWave), lds, st, a);
  };
  using Four = std::integral_constant<int, 4>;
  using All = std::integral_constant<int, kTpgAhead>;
  if (rb == 4) {
    if constexpr (sizeof(T) == 4)
      lds <= kTpgAhead4Lds ? go(Four{}, Four{}) : go(Four{}, All{});
    else
      go(Four{}, Four{});
  } else if (rb == 2) {
    go(std::integral_constant<int, 2>{}, All{});
  } else {
    go(std::integral_constant<int, 1>{}, All{});
  }
  E3_HIP(hipGetLastError());
  if (red && a.pieces > 1) {
    hipLaunchKernelGGL(k_tpg_sum<T>, dim3(blocks_for(rows * a.dout, 256)), dim3(256), 0, st, part, out, rows, a.pieces,
                       a.dout);
    E3_HIP(hipGetLastError());
  }
  return E3_OK;
}
}  // namespace

extern "C" {

e3_status e3_tpg_create(int d_x, int d_y, int d_z, int64_t nnz, const int32_t* i0, const int32_t* i1,
                        const int32_t* i2, const double* val, int y_per_channel, e3_tpg** out) {
  if (!out) return E3_ERR_INVALID_ARG;
  *out = nullptr;
  if (d_x < 1 || d_y < 1 || d_z < 1 || nnz < 0 || nnz > (1 << 24) || (nnz > 0 && (!i0 || !i1 || !i2 || !val)))
    return E3_ERR_INVALID_ARG;
  for (int64_t k = 0; k < nnz; ++k)
    if (i0[k] < 0 || i0[k] >= d_z || i1[k] < 0 || i1[k] >= d_x || i2[k] < 0 || i2[k] >= d_y)
      return E3_ERR_INDEX_OUT_OF_RANGE;
  const bool bsh = !y_per_channel;
  const size_t f = sizeof(float);
  if (tpg_row_lds(d_x, d_y, d_z, bsh, false, f) > kTpgMaxLds || tpg_row_lds(d_z, d_y, d_x, bsh, false, f) > kTpgMaxLds ||
      tpg_row_lds(d_x, d_z, d_y, false, bsh, f) > kTpgMaxLds) {
    g_last_error = "record tensor product: operand rows do not fit the 64 KiB staging limit";
    return E3_ERR_UNSUPPORTED;
  }
  e3_tpg* G = new (std::nothrow) e3_tpg();
  if (!G) return E3_ERR_ALLOC;
  G->d_x = d_x, G->d_y = d_y, G->d_z = d_z, G->ypc = y_per_channel ? 1 : 0;
  std::vector<std::array<int, 3>> kf(nnz), kx(nnz), ky(nnz);
  std::vector<double> v(val, val + nnz);
  for (int64_t k = 0; k < nnz; ++k) {
    kf[k] = {i0[k], i1[k], i2[k]};  // z[i0] from x[i1], y[i2]
    kx[k] = {i1[k], i0[k], i2[k]};  // dx[i1] from dz[i0], y[i2]   (records (i1, i2, i0) of eq. tp-bwd)
    ky[k] = {i2[k], i1[k], i0[k]};  // dy[i2] from x[i1], dz[i0]   (records (i2, i1, i0))
  }
  G->t[0] = tpg_table(d_z, kf, v);
  G->t[1] = tpg_table(d_x, kx, v);
  G->t[2] = tpg_table(d_y, ky, v);
  const e3_status st = tpg_upload(G);
  if (st != E3_OK) {
    delete G;
    return st;
  }
  *out = G;
  return E3_OK;
}

e3_status e3_tpg_destroy(e3_tpg* G) {
  if (!G) return E3_OK;
  if (G->dev) (void)hipFree(G->dev);
  delete G;
  return E3_OK;
}

}  // extern "C"

namespace {
template <class T>
e3_status tpg_fwd(e3_tpg* G, const T* x, const T* y, T* z, int64_t rows, int C, hipStream_t st) {
  if (!G || rows < 0 || C < 1) return E3_ERR_INVALID_ARG;
  if (rows == 0) return E3_OK;
  if (!x || !y || !z) return E3_ERR_INVALID_ARG;
  e3_status s = check_device(G->device, "record tensor-product handle");
  if (s != E3_OK) return s;
  return tpg_run<T>(G, 0, x, G->d_x, y, G->d_y, !G->ypc, z, nullptr, false, rows, C,
                    sizeof(T) == 8 ? "tpg_fwd_f64" : "tpg_fwd", st);
}

size_t tpg_ws(const e3_tpg* G, int64_t rows, int C, size_t elem) {
  return G->ypc ? 0 : align256((size_t)rows * ((C + kWave - 1) / kWave) * G->d_y * elem);
}

template <class T>
e3_status tpg_bwd(e3_tpg* G, const T* x, const T* y, const T* dz, T* dx, T* dy, void* ws, size_t ws_bytes,
                  int64_t rows, int C, hipStream_t st) {
  if (!G || rows < 0 || C < 1) return E3_ERR_INVALID_ARG;
  if (rows == 0) return E3_OK;
  if (!x || !y || !dz || !dx || !dy) return E3_ERR_INVALID_ARG;
  const size_t need = tpg_ws(G, rows, C, sizeof(T));
  if (ws_bytes < need) return E3_ERR_WORKSPACE_TOO_SMALL;
  if (need > 0 && !ws) return E3_ERR_INVALID_ARG;
  e3_status s = check_device(G->device, "record tensor-product handle");
  if (s != E3_OK) return s;
  const bool f64 = sizeof(T) == 8;
  // dx = tensor_product(C^{i1}_{i2 i0}, y, dz)
  if ((s = tpg_run<T>(G, 1, dz, G->d_z, y, G->d_y, !G->ypc, dx, nullptr, false, rows, C,
                      f64 ? "tpg_bwd_dx_f64" : "tpg_bwd_dx", st)) != E3_OK)
    return s;
  // dy = tensor_product(C^{i2}_{i1 i0}, x, dz), summed over the channels when y is shared
  return tpg_run<T>(G, 2, x, G->d_x, dz, G->d_z, false, dy, reinterpret_cast<T*>(ws), !G->ypc, rows, C,
                    f64 ? "tpg_bwd_dy_f64" : "tpg_bwd_dy", st);
}
}  // namespace

extern "C" {

e3_status e3_tpg_fwd(e3_tpg* G, const float* x, const float* y, float* z, int64_t rows, int C, e3_stream stream) {
  return tpg_fwd<float>(G, x, y, z, rows, C, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_tpg_fwd_f64(e3_tpg* G, const double* x, const double* y, double* z, int64_t rows, int C,
                         e3_stream stream) {
  return tpg_fwd<double>(G, x, y, z, rows, C, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_tpg_workspace_size(const e3_tpg* G, int64_t rows, int C, size_t* bwd_bytes) {
  if (!G || rows < 0 || C < 1 || !bwd_bytes) return E3_ERR_INVALID_ARG;
  *bwd_bytes = tpg_ws(G, rows, C, sizeof(double));  // enough for either precision
  return E3_OK;
}

e3_status e3_tpg_bwd(e3_tpg* G, const float* x, const float* y, const float* dz, float* dx, float* dy, void* ws,
                     size_t ws_bytes, int64_t rows, int C, e3_stream stream) {
  return tpg_bwd<float>(G, x, y, dz, dx, dy, ws, ws_bytes, rows, C, reinterpret_cast<hipStream_t>(stream));
}

e3_status e3_tpg_bwd_f64(e3_tpg* G, const double* x, const double* y, const double* dz, double* dx, double* dy,
                         void* ws, size_t ws_bytes, int64_t rows, int C, e3_stream stream) {
  return tpg_bwd<double>(G, x, y, dz, dx, dy, ws, ws_bytes, rows, C, reinterpret_cast<hipStream_t>(stream));
}

}  // extern "C"

// ============================================================ streaming probe
// Instrumentation: the bandwidth HBM sustains for a given read:write mix, with
// the load and store instructions of the sweeps (buffer loads and stores of
// WB bytes per lane at a per-lane offset, with or without the non-temporal
// bit).  Step s reads RU contiguous units of the source and writes WU
// contiguous units of the destination (a unit is 64 lanes x WB bytes), so the
// traffic mix is RU:WU; waves take steps in grid-stride order, so neighbouring
// waves stream neighbouring memory.
// Written only if a wave's sum of loaded values is 3e38, i.e. never for the
// probe's data; its device address is a kernel argument, so that the compiler
// cannot prove the loads feeding that sum unused.
static __device__ __align__(256) float probe_sink[4096];

namespace {

template <int WB, int AUX>
__device__ __forceinline__ float probe_load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  if constexpr (WB == 4) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, AUX));
  } else if constexpr (WB == 8) {
    const f2v t = __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, AUX));
    return t.x + t.y;
  } else {
    const f4v t = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, AUX));
    return (t.x + t.y) + (t.z + t.w);
  }
}

template <int WB, int AUX>
__device__ __forceinline__ void probe_store(__amdgpu_buffer_rsrc_t r, int voff, int soff, float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  if constexpr (WB == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(u, r, voff, soff, AUX);
  } else if constexpr (WB == 8) {
    typedef unsigned u2v __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u2v{u, u}, r, voff, soff, AUX);
  } else {
    typedef unsigned u4v __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(u4v{u, u, u, u}, r, voff, soff, AUX);
  }
}

// Compiled probe shapes (read units, write units, bytes per lane): all loads
// of a step are issued before any is used, as the sweeps issue a row's loads.
#define E3_PROBE_SHAPES(X) \
  X(16, 0, 16) X(16, 0, 8) X(16, 0, 4) X(0, 16, 16) X(0, 16, 8) X(0, 16, 4) X(8, 8, 16) X(14, 1, 8) \
  X(14, 16, 4) X(2, 6, 8) X(8, 2, 8)

template <int WB, int RU, int WU, int LA, int SA>
__global__ __launch_bounds__(256) void k_probe(const char* __restrict__ src, char* __restrict__ dst,
                                               int64_t n_steps, float* __restrict__ sink) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x / kWave);
  // wave index, uniform across the wave (buffer descriptors need scalar bases)
  const int64_t w0 = (int64_t)blockIdx.x * (blockDim.x / kWave) + uniform((int)(threadIdx.x / kWave));
  constexpr int unit = kWave * WB;
  float acc = 0.0f;
  for (int64_t s = w0; s < n_steps; s += nw) {
    if constexpr (RU > 0) {
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<char*>(src) + s * RU * unit, (short)0, RU * unit, 0x00020000);
      float v[RU];
#pragma unroll
      for (int u = 0; u < RU; ++u) v[u] = probe_load<WB, LA>(r, lane * WB, u * unit);
#pragma unroll
      for (int u = 0; u < RU; ++u) acc += v[u];
    }
    if constexpr (WU > 0) {
      const __amdgpu_buffer_rsrc_t r =
          __builtin_amdgcn_make_buffer_rsrc(dst + s * WU * unit, (short)0, WU * unit, 0x00020000);
      const float val = (float)(s & 1023);
#pragma unroll
      for (int u = 0; u < WU; ++u) probe_store<WB, SA>(r, lane * WB, u * unit, val);
    }
  }
  // keeps the loads: never true for finite data below 1e30
  if (acc == 3.0e38f) sink[w0 & 4095] = acc;
}

template <int WB, int RU, int WU>
void probe_launch(const char* src, char* dst, int64_t steps, unsigned flags, int blocks, float* sink,
                  hipStream_t st) {
  const bool nl = flags & 1u, ns = flags & 2u;
  if (nl && ns)
    hipLaunchKernelGGL((k_probe<WB, RU, WU, kNT, kST>), dim3(blocks), dim3(256), 0, st, src, dst, steps, sink);
  else if (nl)
    hipLaunchKernelGGL((k_probe<WB, RU, WU, kNT, 0>), dim3(blocks), dim3(256), 0, st, src, dst, steps, sink);
  else if (ns)
    hipLaunchKernelGGL((k_probe<WB, RU, WU, 0, kST>), dim3(blocks), dim3(256), 0, st, src, dst, steps, sink);
  else
    hipLaunchKernelGGL((k_probe<WB, RU, WU, 0, 0>), dim3(blocks), dim3(256), 0, st, src, dst, steps, sink);
}

bool probe_shape_supported(int ru, int wu, int width) {
#define E3_PROBE_IS(R, W, B) if (ru == R && wu == W && width == B) return true;
  E3_PROBE_SHAPES(E3_PROBE_IS)
#undef E3_PROBE_IS
  return false;
}

std::mutex g_sink_mu;
float* g_sink_ptr[64] = {};

// The current device's copy of probe_sink (looked up once per device).
e3_status sink_of_current_device(float** out) {
  int dev = -1;
  E3_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return E3_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lk(g_sink_mu);
  if (!g_sink_ptr[dev]) {
    void* ptr = nullptr;
    E3_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(probe_sink)));
    g_sink_ptr[dev] = static_cast<float*>(ptr);
  }
  *out = g_sink_ptr[dev];
  return *out ? E3_OK : E3_ERR_HIP;
}
}  // namespace

extern "C" e3_status e3_probe_stream(const void* src, size_t src_bytes, void* dst, size_t dst_bytes,
                                     int read_units, int write_units, int width, unsigned flags,
                                     size_t* bytes_read, size_t* bytes_written, e3_stream stream) {
  if (read_units < 0 || write_units < 0 || read_units + write_units == 0 ||
      (width != 4 && width != 8 && width != 16) || flags > 3u || !bytes_read || !bytes_written)
    return E3_ERR_INVALID_ARG;
  if ((read_units > 0 && (!src || !aligned16(src))) || (write_units > 0 && (!dst || !aligned16(dst))))
    return E3_ERR_INVALID_ARG;
  if (!probe_shape_supported(read_units, write_units, width)) {
    g_last_error = "probe shape not compiled (see E3_PROBE_SHAPES)";
    return E3_ERR_UNSUPPORTED;
  }
  const int64_t unit = (int64_t)kWave * width;
  int64_t steps = INT64_MAX;
  if (read_units > 0) steps = std::min<int64_t>(steps, (int64_t)(src_bytes / (size_t)(unit * read_units)));
  if (write_units > 0) steps = std::min<int64_t>(steps, (int64_t)(dst_bytes / (size_t)(unit * write_units)));
  *bytes_read = (size_t)(steps * unit * read_units);
  *bytes_written = (size_t)(steps * unit * write_units);
  if (steps == 0) return E3_OK;
  // eight waves per SIMD on every compute unit, or fewer when there is less work
  const int blocks = (int)std::min<int64_t>((steps + 3) / 4, 2048);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const char* s = static_cast<const char*>(src);
  char* d = static_cast<char*>(dst);
  float* sink = nullptr;
  const e3_status ss = sink_of_current_device(&sink);
  if (ss != E3_OK) return ss;
  TimedLaunch t_("probe_stream", st);
#define E3_PROBE_GO(R, W, B) \
  if (read_units == R && write_units == W && width == B) probe_launch<B, R, W>(s, d, steps, flags, blocks, sink, st);
  E3_PROBE_SHAPES(E3_PROBE_GO)
#undef E3_PROBE_GO
  E3_HIP(hipGetLastError());
  return E3_OK;
}
