// Hermitian normalization matrices M_ij = sum over points of v_i conj(v_j) of
// C complex amplitudes v (compiled at run time with the model's structure).
//
// The sum over points is a contraction, and it runs on the matrix cores: with
// the real vector w = (Re v, Im v) of R = 2 C entries, M follows from the
// symmetric Gram matrix G = sum w w^T,
//   Re M_ij = G[x_i][x_j] + G[y_i][y_j],  Im M_ij = G[y_i][x_j] - G[x_i][y_j]
// (x, y the real and imaginary entries), accumulated in 16 x 16 tiles on and
// below the diagonal by v_mfma_f64_16x16x4f64 (four points per instruction).
// One pass over the points forms every amplitude once.  The vector passes
// before formed all amplitudes for every two or four rows of M (their 2 x rows
// x C accumulators per lane allowed no more) and took both triangles.
//
// A wave hands its 64 points' vectors over through its own LDS region,
// POINTS at a time: lane p writes column p (rows of POINTS + 1
// doubles: consecutive banks), and the operand of tile t is read as row 16 t +
// l % 16, point 4 s + l / 16 by lane l -- the layout of both MFMA operands,
// since the right one is the transpose (the 16 lanes of one point lie in 16
// bank pairs).  All waves of the grid step through whole groups of 64 points;
// points past the end or outside the region enter as zero vectors.
// A workgroup's four waves are added in a fixed order and it writes one row of
// C (C + 1) / 2 complex sums (i >= j); gram_finalize adds the rows.
#pragma once
#include "device_common.hpp"

namespace fn {

typedef double gram_v4 __attribute__((ext_vector_type(4)));

// Complex sums of a row, index of element (i, j), i >= j.
__host__ __device__ constexpr int gram_count(int C) { return C * (C + 1) / 2; }
__host__ __device__ constexpr int gram_index(int i, int j) { return i * (i + 1) / 2 + j; }

template <int C>
struct Gram {
  static constexpr int R = 2 * C;
  static constexpr int NT = (R + 15) / 16;
  static constexpr int TILES = NT * (NT + 1) / 2;
  static constexpr int RP = 16 * NT;                  // rows with zero padding
  static constexpr int POINTS = RP <= 48 ? 32 : 16;   // points handed over at a time
  static constexpr int LD = POINTS + 1;
  static constexpr int WAVE = RP * LD;                // LDS doubles of a wave
  // the reduction holds two waves' tiles, or one whole Gram matrix
  static constexpr int LDS = kWaves * WAVE > 2 * TILES * 256 ? kWaves * WAVE : 2 * TILES * 256;

  gram_v4 acc[TILES];

  __device__ __forceinline__ void init(double* lds) {
#pragma unroll
    for (int t = 0; t < TILES; ++t) acc[t] = gram_v4{0.0, 0.0, 0.0, 0.0};
    // the padding rows stay zero
    double* w = lds + (threadIdx.x >> 6) * WAVE;
    for (int i = R * LD + (threadIdx.x & 63); i < WAVE; i += 64) w[i] = 0.0;
  }

  // Adds the wave's 64 vectors (re, im: this lane's point).  All 64 lanes call it.
  __device__ __forceinline__ void add(const double (&re)[C], const double (&im)[C], double* lds) {
    const int l = threadIdx.x & 63;
    double* w = lds + (threadIdx.x >> 6) * WAVE;
#pragma unroll
    for (int h = 0; h < 64 / POINTS; ++h) {
      wave_order();  // the reads of the part before come first
      if (l / POINTS == h) {
        const int p = l % POINTS;
#pragma unroll
        for (int k = 0; k < C; ++k) {
          w[k * LD + p] = re[k];
          w[(C + k) * LD + p] = im[k];
        }
      }
      wave_order();
#pragma unroll
      for (int s = 0; s < POINTS / 4; ++s) {
        double op[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) op[t] = w[(16 * t + (l & 15)) * LD + 4 * s + (l >> 4)];
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int b = 0; b <= a; ++b)
            acc[a * (a + 1) / 2 + b] =
                __builtin_amdgcn_mfma_f64_16x16x4f64(op[a], op[b], acc[a * (a + 1) / 2 + b], 0, 0, 0);
      }
    }
  }

  // The workgroup's row.  All threads call it once, after their last add.
  __device__ __forceinline__ void reduce(double* lds, double* __restrict__ row) {
    const int t = threadIdx.x, l = t & 63, wv = t >> 6;
    // waves (0 + 2), (1 + 3), then their sum
    __syncthreads();
    if (wv >= 2) store(lds + (wv - 2) * TILES * 256, l);
    __syncthreads();
    if (wv < 2) load_add(lds + wv * TILES * 256, l);
    __syncthreads();
    if (wv == 1) store(lds, l);
    __syncthreads();
    if (wv == 0) {
      load_add(lds, l);
      // element (i, j) of tile (a, b): lane j + 16 (i % 4), register i / 4
#pragma unroll
      for (int a = 0; a < TILES; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) lds[a * 256 + (4 * v + (l >> 4)) * 16 + (l & 15)] = acc[a][v];
    }
    __syncthreads();
    auto G = [&](int r, int c) {
      const int hi = r > c ? r : c, lo = r > c ? c : r;
      const int a = hi >> 4, b = lo >> 4;
      return lds[(a * (a + 1) / 2 + b) * 256 + (hi & 15) * 16 + (lo & 15)];
    };
    for (int e = t; e < gram_count(C); e += kBlock) {
      int i = 0;
      while (gram_index(i + 1, 0) <= e) ++i;
      const int j = e - gram_index(i, 0);
      row[2 * e] = G(i, j) + G(C + i, C + j);
      row[2 * e + 1] = G(C + i, j) - G(C + j, i);
    }
  }

 private:
  // LDS accesses of the wave's lanes stay in this order (one wave's LDS
  // operations are performed in program order; the fence keeps the compiler's)
  static __device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void store(double* d, int l) const {
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) d[(a * 4 + v) * 64 + l] = acc[a][v];
  }
  __device__ __forceinline__ void load_add(const double* d, int l) {
#pragma unroll
    for (int a = 0; a < TILES; ++a)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[a][v] += d[(a * 4 + v) * 64 + l];
  }
};

}  // namespace fn
