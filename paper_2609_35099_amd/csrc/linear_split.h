// Linear mixing on the bf16 matrix cores at float32 accuracy.
//
// The float32 instruction (v_mfma_f32_16x16x4f32) runs at a sixteenth of the
// bf16 rate.  Here every float32 operand is split into three bf16 terms, each
// the rounding of what the ones before leave: 8 bits each with their signs, so
// that x = h + m + l holds exactly.  A product is eight term products, each
// exact; the one left out, l l, is below 2^-34 of it.  Seven of them (all with
// an m or an l) are summed apart and added on the vector unit, so that a single
// product comes out as the float32 instruction gives it (largest error 6.0e-8,
// L2 2.53e-8; all in one chain, six products: 1.6e-7 and 3.5e-8), and long sums
// come out closer.  Against 64 bits (24,000 nodes, 34 -> 8 blocks of 128,
// float32 instruction -> here): forward 4.5e-7 -> 1.7e-7, dx 2.0e-7 -> 7.3e-8,
// dW 8.2e-7 -> 2.6e-7; sums of 4,096 terms 1.15e-6 -> 4.5e-7, of 8,192 1.62e-6
// -> 6.4e-7; smaller at all of 13 sizes (16 to 192 channels, 64 to 24,000 rows).
//
// Time, same workload (float32 instruction, six products in one chain, here):
// forward 1126, 720, 980 us, dx (the first with a transpose) 1376, 928, 1039 us,
// dW 1258, 969, 1036 us.  Bound by the matrix instructions (0.47 ms at their
// rate) and the splitting (176 vector instructions per step and thread, and 64
// for the sums apart) sharing the issue of each SIMD: two (forward) or three
// workgroups per CU overlap them.  Measured and left: the forward in pairs of
// subtiles on three workgroups 870 us against 921, but 40 against 35 us at 300
// nodes; dx on two 1151 us, dW on two 1083 us (here in that run: 1030, 1012);
// workgroups of 512 threads, 20% slower on 64-wide tiles; loads two steps ahead,
// 2% slower.
//
// A workgroup of four waves takes an RM x BN tile; per 32 of the reduction the
// 256 threads load both operands once (the next step's loads are in flight
// during the instructions), split them and write the terms to LDS as
// [term][row or column][32], which is the operand order of
// v_mfma_f32_16x16x32_bf16: lane l reads 16 bytes of row l % 16 at reduction
// index 8 (l / 16).  The four 16-byte slots of a row are exchanged by row number
// so that the lanes of one pass cover the banks (SpTile).  W takes the
// instruction's A side and the rows the B side, so that a lane owns four
// consecutive output columns.
//
// Infinities and NaNs, operands above 3e26 and sums above 2.8e14 (the scaled
// terms or sums overflow) make the split sums NaN or infinite where float32
// would not: those elements are computed again with the float32 instruction.
// With every operand past the limit: forward 2147 us, dx 2263, dW 2884; with an
// infinity in every 500th node: as without.
#pragma once

namespace {

typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned u2v_ __attribute__((ext_vector_type(2)));
typedef unsigned u4v_ __attribute__((ext_vector_type(4)));

constexpr int kSpThreads = 256;

__device__ __forceinline__ unsigned sp_pack(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{a, b}, bf2v));
}
// The three terms of a and b times kSpScale, packed.  The bf16 instruction
// takes subnormal terms as zero; scaled, every term of every float32 operand
// is normal (unscaled, operands below 1e-33 lost accuracy), and the sums are
// scaled back at the end.
constexpr float kSpScale = 0x1p40f, kSpBack = 0x1p-80f;
__device__ __forceinline__ void sp_split(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  a *= kSpScale, b *= kSpScale;
  h = sp_pack(a, b);
  a -= __uint_as_float(h << 16), b -= __uint_as_float(h & 0xffff0000u);
  m = sp_pack(a, b);
  a -= __uint_as_float(m << 16), b -= __uint_as_float(m & 0xffff0000u);
  l = sp_pack(a, b);
}

// LDS planes of one operand: N rows (or columns) of 32 reduction indexes in
// four 16-byte slots; slot g of a row sits at g ^ f with f = -(row / 4) mod 4,
// so that the lanes of one pass of any access below cover all banks.
template <int N>
struct SpTile {
  unsigned short v[3][N][32];
  __device__ __forceinline__ unsigned short* at(int p, int row, int slot) {
    return &v[p][row][((slot ^ -(row >> 2)) & 3) * 8];
  }
  __device__ __forceinline__ const unsigned short* at(int p, int row, int slot) const {
    return &v[p][row][((slot ^ -(row >> 2)) & 3) * 8];
  }
};

// Thread t's four values at reduction index 4 (t % 8) of rows t / 8 + 32 i.
template <int N>
__device__ __forceinline__ void sp_put_rows(SpTile<N>& s, const f4v (&v)[N / 32]) {
  const int kq = threadIdx.x & 7, row = threadIdx.x >> 3;
#pragma unroll
  for (int i = 0; i < N / 32; ++i) {
    u2v_ h, m, l;
    unsigned a, b, c;
    sp_split(v[i].x, v[i].y, a, b, c);
    h.x = a, m.x = b, l.x = c;
    sp_split(v[i].z, v[i].w, a, b, c);
    h.y = a, m.y = b, l.y = c;
    *reinterpret_cast<u2v_*>(s.at(0, row + 32 * i, kq >> 1) + 4 * (kq & 1)) = h;
    *reinterpret_cast<u2v_*>(s.at(1, row + 32 * i, kq >> 1) + 4 * (kq & 1)) = m;
    *reinterpret_cast<u2v_*>(s.at(2, row + 32 * i, kq >> 1) + 4 * (kq & 1)) = l;
  }
}

// Thread t's N / 8 values of column t % N at reduction index (t / N) N / 8 on.
template <int N>
__device__ __forceinline__ void sp_put_cols(SpTile<N>& s, const float (&v)[N / 8]) {
  const int col = threadIdx.x % N, k0 = (threadIdx.x / N) * (N / 8);
#pragma unroll
  for (int q = 0; q < N / 64; ++q) {
    u4v_ h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned a, b, c;
      sp_split(v[8 * q + 2 * e], v[8 * q + 2 * e + 1], a, b, c);
      h[e] = a, m[e] = b, l[e] = c;
    }
    *reinterpret_cast<u4v_*>(s.at(0, col, k0 / 8 + q)) = h;
    *reinterpret_cast<u4v_*>(s.at(1, col, k0 / 8 + q)) = m;
    *reinterpret_cast<u4v_*>(s.at(2, col, k0 / 8 + q)) = l;
  }
}

// The wave's part of the tile: 16 RS rows from row0, 64 columns from col0.
template <int RM, int BN>
struct SpWave {
  static constexpr int WC = BN / 64, WR = 4 / WC, RS = RM / WR / 16;
  static_assert(RS >= 1);
  int row0, col0, li, g;
  f4v acc[RS][4];
  __device__ __forceinline__ SpWave() {
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    row0 = (w / WC) * 16 * RS, col0 = (w % WC) * 64, li = lane & 15, g = lane >> 4;
#pragma unroll
    for (int s = 0; s < RS; ++s)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[s][c] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
  }
  // One step of 32: X are the rows' terms, Y the columns'.  The products with a
  // lower term are summed on their own, smallest first, and added to the rest by
  // the vector unit: they are a 256th of the sum and lose nothing there, and the
  // product of the two first terms, which is exact, meets them in one rounding
  // to nearest (the instruction's own additions err by up to twice as much).
  // APART: the products of the first terms are summed apart from the running
  // sum too, which keeps long reductions accurate.
  // SP subtiles at a time; fewer take fewer registers, read the columns' terms
  // more often and make a longer chain.
  template <bool APART, int SP>
  __device__ __forceinline__ void step(const SpTile<RM>& X, const SpTile<BN>& Y) {
    constexpr f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int PY[7] = {2, 1, 2, 0, 1, 1, 0}, PX[7] = {1, 2, 0, 2, 1, 0, 1};
#pragma unroll
    for (int s0 = 0; s0 < RS; s0 += SP) {
      bf8v x[3][SP];
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int s = 0; s < SP; ++s) x[p][s] = *reinterpret_cast<const bf8v*>(X.at(p, row0 + 16 * (s0 + s) + li, g));
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        bf8v y[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) y[p] = *reinterpret_cast<const bf8v*>(Y.at(p, col0 + 16 * c + li, g));
        f4v lo[SP];
#pragma unroll
        for (int s = 0; s < SP; ++s) lo[s] = zero;
#pragma unroll
        for (int t = 0; t < 7; ++t)
#pragma unroll
          for (int s = 0; s < SP; ++s)
            lo[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[PY[t]], x[PX[t]][s], lo[s], 0, 0, 0);
#pragma unroll
        for (int s = 0; s < SP; ++s) {
          f4v& sum = acc[s0 + s][c];
          const f4v hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[0], x[0][s], APART ? zero : sum, 0, 0, 0);
          sum = APART ? sum + hi : hi;
        }
#pragma unroll
        for (int s = 0; s < SP; ++s) acc[s0 + s][c] += lo[s];
        // the compiler would start the next columns early and spill
        if (!APART && SP < RS) __builtin_amdgcn_sched_barrier(0);
      }
      if (SP < RS) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");  // the next subtiles read the columns' terms again
      }
    }
  }
  // The results: the sums scaled back, and in the place of one that is not
  // finite what the float32 instruction gives, so that an element depends on its
  // own row and column alone.  row(s, k), col(c, k): the operands at reduction
  // indexes k + 4 g .. + 3 of the lane's row of subtile s and column of subtile c.
  template <class FR, class FC>
  __device__ __forceinline__ void finish(int kn, FR&& row, FC&& col) {
    constexpr int SP = RS < 2 ? 1 : 2;
#pragma unroll
    for (int s0 = 0; s0 < RS; s0 += SP) {
      float z = 0.0f;
#pragma unroll
      for (int s = s0; s < s0 + SP; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) z += acc[s][c][r] * 0.0f;
      if (__ballot(z != 0.0f) == 0) {  // no NaN in any lane: all finite
#pragma unroll
        for (int s = s0; s < s0 + SP; ++s)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[s][c] *= kSpBack;
        continue;
      }
      f4v t[SP][4];
#pragma unroll
      for (int s = 0; s < SP; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) t[s][c] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
      for (int k = 0; k < kn; k += 16) {
        f4v x[SP], y[4];
#pragma unroll
        for (int s = 0; s < SP; ++s) x[s] = row(s0 + s, k);
#pragma unroll
        for (int c = 0; c < 4; ++c) y[c] = col(c, k);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int s = 0; s < SP; ++s)
              t[s][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(y[c][e], x[s][e], t[s][c], 0, 0, 0);
      }
#pragma unroll
      for (int s = 0; s < SP; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v = acc[s0 + s][c][r];
            acc[s0 + s][c][r] = v * 0.0f == 0.0f ? v * kSpBack : t[s][c][r];
          }
    }
  }
};

// v / R and v % R by a multiplication and a correction: with mul = 2^32 / R
// rounded up, the product's high half is at most one too large for any v < 2^31.
struct SpDiv {
  int R;
  unsigned mul;  // 0 for R = 1
  __device__ __forceinline__ explicit SpDiv(int R_) : R(R_), mul(0xffffffffu / R_ + 1) {}
  __device__ __forceinline__ int operator()(int v, int& rem) const {
    const int q = mul ? (int)__umulhi((unsigned)v, mul) : v, m = v - q * R;
    rem = m < 0 ? m + R : m;
    return m < 0 ? q - 1 : q;
  }
};

// Rows r0 + d of a tile as (node, component of R).
struct SpRows {
  int64_t node0;
  int m0, last;
  SpDiv div;
  __device__ __forceinline__ SpRows(int64_t r0, int64_t NR, int R) : div(R) {
    node0 = r0 / R, m0 = (int)(r0 - node0 * R);
    last = NR - r0 < 1024 ? (int)(NR - r0) - 1 : 1023;  // rows past the end become the last one
  }
  // offset of row d's component row in units of rows of a tensor with D per node, from node0
  __device__ __forceinline__ int at(int d, int D) const {
    int m;
    const int q = div(m0 + imin(d, last), m);
    return q * D + m;
  }
};

// Destination rows = sum over the job's sources and k of src[row, k] B[k, col].
// TB: a W slice is [col][k] (rows of C_src, 16-byte aligned), else [k][col]
// (rows of C_dst).
template <int RM, int BN, bool TB>
__global__ __launch_bounds__(kSpThreads, TB ? 3 : 2) void k_lin_gemm(LinArgs a) {
  __shared__ __align__(16) SpTile<RM> sX;
  __shared__ __align__(16) SpTile<BN> sW;
  const int64_t block = block_id();
  if (block >= a.first[a.njobs]) return;
  const int unit = (int)block;
  int lo = 0, hi = a.njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.first[mid] <= unit) lo = mid; else hi = mid - 1;
  }
  const LinJob jb = a.jobs[lo];
  const ConstPtr<LinSrc> srcs = (ConstPtr<LinSrc>)a.srcs + jb.src_first;
  const int u = unit - a.first[lo];
  const int col0 = (u % a.slabs) * BN;
  const int64_t r0 = (int64_t)(u / a.slabs) * RM, NR = a.n * jb.R;
  const int tid = threadIdx.x, kq = tid & 7, hh = kq >> 2;
  // rows past the end load the last row, columns past C_dst the last column;
  // their results are not stored
  unsigned xp[RM / 32];  // units of 16 channels: below 2^32 for any layout
  const SpRows rows(r0, NR, jb.R);
  const float* src0 = a.src + rows.node0 * a.D_src * a.C_src;
#pragma unroll
  for (int i = 0; i < RM / 32; ++i)
    xp[i] = (unsigned)rows.at((tid >> 3) + 32 * i, a.D_src) * (unsigned)(a.C_src / 16);
  // the reduction runs over halves of 16 (C_src is a multiple of 16), two per step
  const int hs = a.C_src / 16, nh = jb.nsrc * hs, nsteps = (nh + 1) / 2;
  f4v xv[RM / 32];
  float wv[TB ? 1 : BN / 8];
  f4v wt[TB ? BN / 32 : 1];
  auto load = [&](int st) {
    st = imin(st, nsteps - 1);  // unconditional loads: the waits count exactly
    const int h0 = 2 * st, h1 = h0 + 1 < nh ? h0 + 1 : h0;  // uniform
    const int t0 = h0 / hs, t1 = h1 / hs, k0 = (h0 - t0 * hs) * 16, k1 = (h1 - t1 * hs) * 16;
    const int x0 = srcs[t0].row * a.C_src + k0, x1 = srcs[t1].row * a.C_src + k1;
    const float* sp = src0 + ((hh ? x1 : x0) + 4 * (kq & 3));
#pragma unroll
    for (int i = 0; i < RM / 32; ++i) xv[i] = *reinterpret_cast<const f4v*>(sp + ((uint64_t)xp[i] << 4));
    const int64_t w0 = srcs[t0].w_off, w1 = srcs[t1].w_off;
    if constexpr (TB) {
      const float* wp = a.W + (hh ? w1 + k1 : w0 + k0) + 4 * (kq & 3);
#pragma unroll
      for (int i = 0; i < BN / 32; ++i) {
        const int c = imin(col0 + (tid >> 3) + 32 * i, a.C_dst - 1);
        wt[i] = *reinterpret_cast<const f4v*>(wp + (unsigned)(c * a.C_src));
      }
    } else {
      // thread's N / 8 reduction indexes: in half 0 or 1, uniform per wave
      const int kk = uniform(tid / BN) * (BN / 8), hb = kk >> 4;
      const float* wp = a.W + (hb ? w1 : w0) + (int64_t)((hb ? k1 : k0) + (kk & 15)) * a.C_dst;
      const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float*>(wp), (short)0, (BN / 8) * a.C_dst * 4, 0x00020000);
      const int voff = imin(col0 + tid % BN, a.C_dst - 1) * 4;
#pragma unroll
      for (int e = 0; e < BN / 8; ++e)
        wv[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, voff, e * a.C_dst * 4, 0));
    }
  };
  // Subtiles at a time: the forward (many sources) all of them on two workgroups
  // per CU, dx (few) in pairs on three.
  constexpr int kSub = TB && SpWave<RM, BN>::RS > 2 ? 2 : SpWave<RM, BN>::RS;
  SpWave<RM, BN> w;
  if (nsteps > 0) load(0);
  for (int st = 0; st < nsteps; ++st) {
    // the missing half of an odd count is cleared here, not at the load, which
    // would wait for it
    if (2 * st + 1 >= nh && hh)
#pragma unroll
      for (int i = 0; i < RM / 32; ++i) xv[i] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    sp_put_rows<RM>(sX, xv);
    if constexpr (TB) sp_put_rows<BN>(sW, wt);
    else sp_put_cols<BN>(sW, wv);
    __syncthreads();
    load(st + 1);
    w.template step<false, kSub>(sX, sW);
    __syncthreads();
  }
  w.finish(jb.nsrc * a.C_src,
           [&](int s, int k) {
             const int t = k / a.C_src, d = w.row0 + 16 * s + w.li;
             return *reinterpret_cast<const f4v*>(src0 + ((int64_t)rows.at(d, a.D_src) + srcs[t].row) * a.C_src +
                                                  (k - t * a.C_src + 4 * w.g));
           },
           [&](int c, int k) {
             const int t = k / a.C_src, kk = k - t * a.C_src + 4 * w.g;
             const int col = imin(col0 + w.col0 + 16 * c + w.li, a.C_dst - 1);
             const float* p = a.W + srcs[t].w_off;
             if constexpr (TB) return *reinterpret_cast<const f4v*>(p + ((int64_t)col * a.C_src + kk));
             f4v v;
#pragma unroll
             for (int e = 0; e < 4; ++e) v[e] = p[(int64_t)(kk + e) * a.C_dst + col];
             return v;
           });
  float* dst0 = a.dst + (rows.node0 * a.D_dst + jb.dst_row) * a.C_dst;
  // lane l of acc[s][c]: row l % 16 of subtile s, columns 4 (l / 16) .. +3 of subtile c
#pragma unroll
  for (int s = 0; s < SpWave<RM, BN>::RS; ++s) {
    const int d = w.row0 + 16 * s + w.li;
    if (d > rows.last) continue;
    float* dp = dst0 + (int64_t)rows.at(d, a.D_dst) * a.C_dst + col0 + w.col0 + 4 * w.g;
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (col0 + w.col0 + 16 * c + 4 * w.g < a.C_dst) *reinterpret_cast<f4v*>(dp + 16 * c) = w.acc[s][c];
  }
}

// dW partials of one (pair, row chunk, RM x BN tile of W): the reduction runs
// over the chunk's rows, so both operands are staged by columns.
template <int RM, int BN>
__global__ __launch_bounds__(kSpThreads, 3) void k_lin_dw(LinDwArgs a) {
  __shared__ __align__(16) SpTile<RM> sX;
  __shared__ __align__(16) SpTile<BN> sD;
  const int per = kLinChunks * a.ktiles * a.jtiles;
  const int64_t block = block_id();
  const int p = (int)(block / per), u = (int)(block % per);
  if (p >= a.npairs) return;
  const int chunk = u / (a.ktiles * a.jtiles), kc0 = (u / a.jtiles) % a.ktiles * RM, jc0 = u % a.jtiles * BN;
  const LinPair pr = a.pairs[p];
  const int R = pr.R, tid = threadIdx.x;
  const int64_t NR = a.n * R;
  const int64_t rpc = ((NR + kLinChunks - 1) / kLinChunks + 15) / 16 * 16;  // rows per chunk, a multiple of 16
  const int64_t rb = chunk * rpc < NR ? chunk * rpc : NR, re = rb + rpc < NR ? rb + rpc : NR;
  const int nrows = (int)(re - rb), nsteps = (nrows + 31) / 32;
  // Columns past C_in / C_out read the last one; their results are not stored.
  // A thread's N / 8 rows of a step are uniform per wave; rows past the end
  // load the last row and are cleared.
  const unsigned xcol = imin(kc0 + tid % RM, a.C_in - 1), dcol = imin(jc0 + tid % BN, a.C_out - 1);
  float xv[RM / 8], dv[BN / 8];
  // Row offsets from the node of the step's first row, a row per lane (they
  // repeat every 16 lanes), handed out by v_readlane: in units of 16 channels,
  // which stay below 2^31 for any layout (64 blocks of up to 1,999 rows, 4,096
  // channels, 32 nodes), where bytes would not.
  const int64_t node0 = rb / R;
  const int m0 = (int)(rb - node0 * R), lane16 = tid & 15;
  const SpDiv div(R);
  auto load = [&](int st) {
    st = imin(st, nsteps - 1);  // unconditional loads: the waits count exactly
    int m1;
    const int q1 = div(m0 + 32 * st, m1);
    const float* x0 = a.x + ((node0 + q1) * a.D_in + pr.src_row) * a.C_in;
    const float* d0 = a.dout + ((node0 + q1) * a.D_out + pr.dst_row) * a.C_out;
    auto rows = [&](auto& v, const float* base, int D, int C, unsigned col, int k0) {
      constexpr int cnt = sizeof(v) / sizeof(v[0]);
      int m;
      const int q = div(m1 + imin(k0 + lane16, nrows - 1 - 32 * st), m);
      const int off = (q * D + m) * (C / 16);
#pragma unroll
      for (int e = 0; e < cnt; ++e) v[e] = (base + ((uint64_t)(unsigned)__builtin_amdgcn_readlane(off, e) << 4))[col];
    };
    rows(xv, x0, a.D_in, a.C_in, xcol, uniform(tid / RM) * (RM / 8));
    rows(dv, d0, a.D_out, a.C_out, dcol, uniform(tid / BN) * (BN / 8));
  };
  SpWave<RM, BN> w;
  if (nsteps > 0) load(0);
  for (int st = 0; st < nsteps; ++st) {
    const int left = nrows - 32 * st - uniform(tid / RM) * (RM / 8);
    if (left < RM / 8)  // clearing one side of the product is enough
#pragma unroll
      for (int e = 0; e < RM / 8; ++e)
        if (e >= left) xv[e] = 0.0f;
    sp_put_cols<RM>(sX, xv);
    sp_put_cols<BN>(sD, dv);
    __syncthreads();
    load(st + 1);
    w.template step<true, SpWave<RM, BN>::RS < 2 ? 1 : 2>(sX, sD);
    __syncthreads();
  }
  auto operand = [&](const float* p, int D, int row, int C, int ch, int k) {
    f4v v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = k + 4 * w.g + e;  // rows past the end: zero
      const int64_t r = rb + imin(i, nrows - 1);
      const float u = p[((r / R) * D + row + r % R) * C + imin(ch, C - 1)];
      v[e] = i < nrows ? u : 0.0f;
    }
    return v;
  };
  w.finish(nrows,
           [&](int s, int k) { return operand(a.x, a.D_in, pr.src_row, a.C_in, kc0 + w.row0 + 16 * s + w.li, k); },
           [&](int c, int k) { return operand(a.dout, a.D_out, pr.dst_row, a.C_out, jc0 + w.col0 + 16 * c + w.li, k); });
  float* out = a.dWp + ((int64_t)p * kLinChunks + chunk) * a.C_in * a.C_out;
#pragma unroll
  for (int s = 0; s < SpWave<RM, BN>::RS; ++s) {
    const int k = kc0 + w.row0 + 16 * s + w.li;
    if (k >= a.C_in) continue;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int j = jc0 + w.col0 + 16 * c + 4 * w.g;
      if (j < a.C_out) *reinterpret_cast<f4v*>(out + (int64_t)k * a.C_out + j) = w.acc[s][c];
    }
  }
}

}  // namespace
