// Three-stage line FFT (L = R1 R2 R3) with more threads per line and fewer
// elements per thread than the two-stage version; used by the N0 passes and
// the long lines of k_plane, which hold a residual or an accumulator beside
// the line.
//
// Forward, with Q = R2 R3:
//   stage 1: butterfly b in [0, Q):        x[b + Q n1]            -> Y1[b][k1]  * W_L^{b k1}
//   stage 2: butterfly (k1, b2):            Y1[b2 + R3 n2][k1]     -> Y2[k1][b2][k2] * W_Q^{b2 k2}
//   stage 3: butterfly (k1, k2):            Y2[k1][b2][k2] over b2 -> X[k1 + R1 (k2 + R2 k3)]
// Layout A (natural): thread t holds x[(t + T u) + Q n1], e = u R1 + n1.
// Layout B (spectral): thread t holds X[k1 + R1 (k2 + R2 k3)] with
// (k1, k2) = (g % R1, g / R1), g = t + T z, e = z R3 + k3.
// The inverse runs the stages backwards with conjugate twiddles (B -> A).
#pragma once
#include <type_traits>

#include "fg_fft.hpp"

namespace fg {

template <int L> struct Line3Shape;
template <> struct Line3Shape<256> {
  static constexpr int R1 = 8, R2 = 8, R3 = 4, T = 32;
};
template <> struct Line3Shape<128> {
  static constexpr int R1 = 4, R2 = 4, R3 = 8, T = 16;
};
template <> struct Line3Shape<96> {
  static constexpr int R1 = 4, R2 = 4, R3 = 6, T = 8;
};
template <> struct Line3Shape<512> {
  static constexpr int R1 = 8, R2 = 8, R3 = 8, T = 64;
};

// CPT adjacent columns of one LDS row position in one access (two
// single-precision complex values: one 16-byte access, the same bank pattern
// as one double-precision column).
template <int CPT, typename C> __device__ __forceinline__ void lds_put(C* p, const C (&x)[CPT]) {
  if constexpr (CPT == 2) {
    static_assert(sizeof(C) == 8, "column pairs in single precision");
    *reinterpret_cast<float4*>(p) = make_float4(x[0].x, x[0].y, x[CPT - 1].x, x[CPT - 1].y);
  } else {
    *p = x[0];
  }
}
template <int CPT, typename C> __device__ __forceinline__ void lds_get(const C* p, C (&x)[CPT]) {
  if constexpr (CPT == 2) {
    const float4 w = *reinterpret_cast<const float4*>(p);
    x[0] = mk<C>(w.x, w.y);
    x[CPT - 1] = mk<C>(w.z, w.w);
  } else {
    x[0] = *p;
  }
}

template <int L> struct Line3 {
  static constexpr int R1 = Line3Shape<L>::R1, R2 = Line3Shape<L>::R2, R3 = Line3Shape<L>::R3;
  static constexpr int T = Line3Shape<L>::T;
  static constexpr int Q = R2 * R3;
  static constexpr int U1 = Q / T, U2 = R1 * R3 / T, U3 = R1 * R2 / T;
  static constexpr int E = L / T;
  static_assert(U1 * T == Q && U2 * T == R1 * R3 && U3 * T == R1 * R2, "thread split");
  static_assert(U1 * R1 == E && U2 * R2 == E && U3 * R3 == E, "element split");
  __device__ __forceinline__ static int idxA(int t, int e) { return t + T * (e / R1) + Q * (e % R1); }
  __device__ __forceinline__ static int idxB(int t, int e) {
    const int g = t + T * (e / R3);
    return (g % R1) + R1 * ((g / R1) + R2 * (e % R3));
  }
  // LDS positions of the intermediate arrays
  __device__ __forceinline__ static int pos1(int b, int k1) { return b * R1 + k1; }
  __device__ __forceinline__ static int pos2(int k1, int b2, int k2) { return (k2 * R3 + b2) * R1 + k1; }

  template <bool INV, typename C, bool WAVE = false>
  __device__ __forceinline__ static void fwd(C (&v)[E], C* lds, int ls, int t, const C* tw) {
#pragma unroll
    for (int u = 0; u < U1; ++u) {
      const int b = t + T * u;
      Dft<R1, 1, INV, C>::run(v + u * R1);
#pragma unroll
      for (int k1 = 1; k1 < R1; ++k1) v[u * R1 + k1] = twiddle_tab<INV>(v[u * R1 + k1], tw, (b * k1) % L);
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) lds[pos1(b, k1) * ls] = v[u * R1 + k1];
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int w = 0; w < U2; ++w) {
      const int g = t + T * w;
      const int k1 = g % R1, b2 = g / R1;
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) v[w * R2 + n2] = lds[pos1(b2 + R3 * n2, k1) * ls];
      Dft<R2, 1, INV, C>::run(v + w * R2);
#pragma unroll
      for (int k2 = 1; k2 < R2; ++k2) v[w * R2 + k2] = twiddle_tab<INV>(v[w * R2 + k2], tw, (R1 * b2 * k2) % L);
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int w = 0; w < U2; ++w) {
      const int g = t + T * w;
      const int k1 = g % R1, b2 = g / R1;
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) lds[pos2(k1, b2, k2) * ls] = v[w * R2 + k2];
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int z = 0; z < U3; ++z) {
      const int g = t + T * z;
      const int k1 = g % R1, k2 = g / R1;
#pragma unroll
      for (int b2 = 0; b2 < R3; ++b2) v[z * R3 + b2] = lds[pos2(k1, b2, k2) * ls];
      Dft<R3, 1, INV, C>::run(v + z * R3);
    }
    lds_sync<WAVE>();
  }

  template <typename C, bool WAVE = false>
  __device__ __forceinline__ static void inv(C (&v)[E], C* lds, int ls, int t, const C* tw) {
#pragma unroll
    for (int z = 0; z < U3; ++z) {
      const int g = t + T * z;
      const int k1 = g % R1, k2 = g / R1;
      Dft<R3, 1, true, C>::run(v + z * R3);  // over k3 -> b2
#pragma unroll
      for (int b2 = 0; b2 < R3; ++b2) {
        C a = v[z * R3 + b2];
        if (b2 != 0 && k2 != 0) a = twiddle_tab<true>(a, tw, (R1 * b2 * k2) % L);
        lds[pos2(k1, b2, k2) * ls] = a;
      }
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int w = 0; w < U2; ++w) {
      const int g = t + T * w;
      const int k1 = g % R1, b2 = g / R1;
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) v[w * R2 + k2] = lds[pos2(k1, b2, k2) * ls];
      Dft<R2, 1, true, C>::run(v + w * R2);  // over k2 -> n2
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int w = 0; w < U2; ++w) {
      const int g = t + T * w;
      const int k1 = g % R1, b2 = g / R1;
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) {
        const int b = b2 + R3 * n2;
        C a = v[w * R2 + n2];
        if (k1 != 0) a = twiddle_tab<true>(a, tw, (b * k1) % L);
        lds[pos1(b, k1) * ls] = a;
      }
    }
    lds_sync<WAVE>();
#pragma unroll
    for (int u = 0; u < U1; ++u) {
      const int b = t + T * u;
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) v[u * R1 + k1] = lds[pos1(b, k1) * ls];
      Dft<R1, 1, true, C>::run(v + u * R1);  // over k1 -> n1
    }
    lds_sync<WAVE>();
  }

  // fwd and inv of CPT adjacent columns together (lds points at the first
  // column, which is CPT-aligned; one CPT-wide LDS access per position).
  template <bool INV, int CPT, typename C>
  __device__ __forceinline__ static void fwd_cols(C (&v)[CPT][E], C* lds, int ls, int t, const C* tw) {
    if constexpr (CPT == 1) {
      fwd<INV>(v[0], lds, ls, t, tw);
    } else {
#pragma unroll
      for (int u = 0; u < U1; ++u) {
        const int b = t + T * u;
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          Dft<R1, 1, INV, C>::run(v[c] + u * R1);
#pragma unroll
          for (int k1 = 1; k1 < R1; ++k1) v[c][u * R1 + k1] = twiddle_tab<INV>(v[c][u * R1 + k1], tw, (b * k1) % L);
        }
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1) {
          C x[CPT];
#pragma unroll
          for (int c = 0; c < CPT; ++c) x[c] = v[c][u * R1 + k1];
          lds_put<CPT>(lds + pos1(b, k1) * ls, x);
        }
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < U2; ++w) {
        const int g = t + T * w;
        const int k1 = g % R1, b2 = g / R1;
#pragma unroll
        for (int n2 = 0; n2 < R2; ++n2) {
          C x[CPT];
          lds_get<CPT>(lds + pos1(b2 + R3 * n2, k1) * ls, x);
#pragma unroll
          for (int c = 0; c < CPT; ++c) v[c][w * R2 + n2] = x[c];
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
          Dft<R2, 1, INV, C>::run(v[c] + w * R2);
#pragma unroll
          for (int k2 = 1; k2 < R2; ++k2)
            v[c][w * R2 + k2] = twiddle_tab<INV>(v[c][w * R2 + k2], tw, (R1 * b2 * k2) % L);
        }
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < U2; ++w) {
        const int g = t + T * w;
        const int k1 = g % R1, b2 = g / R1;
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) {
          C x[CPT];
#pragma unroll
          for (int c = 0; c < CPT; ++c) x[c] = v[c][w * R2 + k2];
          lds_put<CPT>(lds + pos2(k1, b2, k2) * ls, x);
        }
      }
      __syncthreads();
#pragma unroll
      for (int z = 0; z < U3; ++z) {
        const int g = t + T * z;
        const int k1 = g % R1, k2 = g / R1;
#pragma unroll
        for (int b2 = 0; b2 < R3; ++b2) {
          C x[CPT];
          lds_get<CPT>(lds + pos2(k1, b2, k2) * ls, x);
#pragma unroll
          for (int c = 0; c < CPT; ++c) v[c][z * R3 + b2] = x[c];
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) Dft<R3, 1, INV, C>::run(v[c] + z * R3);
      }
      __syncthreads();
    }
  }

  template <int CPT, typename C>
  __device__ __forceinline__ static void inv_cols(C (&v)[CPT][E], C* lds, int ls, int t, const C* tw) {
    if constexpr (CPT == 1) {
      inv(v[0], lds, ls, t, tw);
    } else {
#pragma unroll
      for (int z = 0; z < U3; ++z) {
        const int g = t + T * z;
        const int k1 = g % R1, k2 = g / R1;
#pragma unroll
        for (int c = 0; c < CPT; ++c) Dft<R3, 1, true, C>::run(v[c] + z * R3);  // over k3 -> b2
#pragma unroll
        for (int b2 = 0; b2 < R3; ++b2) {
          C x[CPT];
#pragma unroll
          for (int c = 0; c < CPT; ++c) {
            x[c] = v[c][z * R3 + b2];
            if (b2 != 0 && k2 != 0) x[c] = twiddle_tab<true>(x[c], tw, (R1 * b2 * k2) % L);
          }
          lds_put<CPT>(lds + pos2(k1, b2, k2) * ls, x);
        }
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < U2; ++w) {
        const int g = t + T * w;
        const int k1 = g % R1, b2 = g / R1;
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) {
          C x[CPT];
          lds_get<CPT>(lds + pos2(k1, b2, k2) * ls, x);
#pragma unroll
          for (int c = 0; c < CPT; ++c) v[c][w * R2 + k2] = x[c];
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) Dft<R2, 1, true, C>::run(v[c] + w * R2);  // over k2 -> n2
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < U2; ++w) {
        const int g = t + T * w;
        const int k1 = g % R1, b2 = g / R1;
#pragma unroll
        for (int n2 = 0; n2 < R2; ++n2) {
          const int b = b2 + R3 * n2;
          C x[CPT];
#pragma unroll
          for (int c = 0; c < CPT; ++c) {
            x[c] = v[c][w * R2 + n2];
            if (k1 != 0) x[c] = twiddle_tab<true>(x[c], tw, (b * k1) % L);
          }
          lds_put<CPT>(lds + pos1(b, k1) * ls, x);
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U1; ++u) {
        const int b = t + T * u;
#pragma unroll
        for (int k1 = 0; k1 < R1; ++k1) {
          C x[CPT];
          lds_get<CPT>(lds + pos1(b, k1) * ls, x);
#pragma unroll
          for (int c = 0; c < CPT; ++c) v[c][u * R1 + k1] = x[c];
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) Dft<R1, 1, true, C>::run(v[c] + u * R1);  // over k1 -> n1
      }
      __syncthreads();
    }
  }
};

// The two-stage transform behind the same interface.
template <int L> struct Line2Ops {
  using LS = Line<L>;
  static constexpr int T = LS::T, E = LS::E;
  __device__ __forceinline__ static int idxA(int t, int e) { return LS::idxA(t, e); }
  __device__ __forceinline__ static int idxB(int t, int e) { return LS::idxB(t, e); }
  template <bool INV, typename C, bool WAVE = false>
  __device__ __forceinline__ static void fwd(C (&v)[E], C* lds, int ls, int t, const C* tw) {
    line_fft_AB<L, INV, C, WAVE>(v, lds, ls, t, tw);
  }
  template <typename C, bool WAVE = false>
  __device__ __forceinline__ static void inv(C (&v)[E], C* lds, int ls, int t, const C* tw) {
    line_ifft_BA<L, C, WAVE>(v, lds, ls, t, tw);
  }
  // columns one after the other (one element per LDS access)
  template <bool INV, int CPT, typename C>
  __device__ __forceinline__ static void fwd_cols(C (&v)[CPT][E], C* lds, int ls, int t, const C* tw) {
#pragma unroll
    for (int c = 0; c < CPT; ++c) fwd<INV>(v[c], lds + c, ls, t, tw);
  }
  template <int CPT, typename C>
  __device__ __forceinline__ static void inv_cols(C (&v)[CPT][E], C* lds, int ls, int t, const C* tw) {
#pragma unroll
    for (int c = 0; c < CPT; ++c) inv(v[c], lds + c, ls, t, tw);
  }
};

// Line transform used by the fused N0 passes.
template <int L> struct ZLineSel {
  using type = Line2Ops<L>;
};
template <> struct ZLineSel<256> {
  using type = Line3<256>;
};
template <> struct ZLineSel<128> {
  using type = Line3<128>;
};
template <> struct ZLineSel<96> {
  using type = Line3<96>;
};
template <> struct ZLineSel<512> {
  using type = Line3<512>;
};
template <int L> using ZLine = typename ZLineSel<L>::type;
// Line of the N0 pass of the CG (k_n0): ZLine, except the two-stage 16 x 16
// line in single precision at L = 256 (one column per thread there).
template <typename R, int L> struct ZGradSel {
  using type = ZLine<L>;
};
template <> struct ZGradSel<float, 256> {
  using type = Line2Ops<256>;
};

template <typename R, int L>
__global__ void __launch_bounds__(256)
k_fft_z_proj(R* data, int N1, int M, int B, SpecTables<R> tb, R scale, Skip skip, int kymajor) {
  using C = cplx<R>;
  using LS = ZLine<L>;
  extern __shared__ __align__(16) char smem_raw[];
  C* lds = reinterpret_cast<C*>(smem_raw);
  C* stw = lds + L * B;
  R* scz = reinterpret_cast<R*>(stw + L);
  R* ssz = scz + L;
  if (skip(blockIdx.z)) return;
  for (int k = threadIdx.x; k < L; k += blockDim.x) {
    stw[k] = tb.tw0[k];
    scz[k] = tb.cz[k];
    ssz[k] = tb.sz[k];
  }
  __syncthreads();
  const int col = threadIdx.x % B;
  const int t = threadIdx.x / B;
  // workgroup order: kx tiles fastest (grid M/B x N1), or ky fastest
  // (grid N1 x M/B: consecutive workgroups then sit 16 M bytes apart
  // instead of 16 B bytes, spreading concurrent accesses over the plane)
  const int kx = (kymajor ? blockIdx.y : blockIdx.x) * B + col;
  const int ky = kymajor ? blockIdx.x : blockIdx.y;
  const int i = blockIdx.z;
  const long plane = (long)N1 * M;
  const long comp = (long)L * plane;
  // (ky, kx) factors of the rotated vector: r = (sz cy cx, cz sy cx, cz cy sx)
  const R cy = tb.cy[ky], sy = tb.sy[ky], cx = tb.cx[kx], sx = tb.sx[kx];
  const R fx0 = cy * cx, fx1 = sy * cx, fx2 = cy * sx;
  C* base = reinterpret_cast<C*>(data) + (long)ky * M + kx;
  C acc[LS::E];
#pragma unroll
  for (int e = 0; e < LS::E; ++e) acc[e] = mk<C>(R(0), R(0));
#pragma unroll 1
  for (int l = 0; l < 3; ++l) {
    const C* src = base + (3 * i + l) * comp;
    C v[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) v[e] = src[LS::idxA(t, e) * plane];
    LS::template fwd<false>(v, lds + col, B, t, stw);
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e);
      const R rl = (l == 0) ? ssz[kz] * fx0 : scz[kz] * (l == 1 ? fx1 : fx2);
      acc[e] = mk<C>(acc[e].x + v[e].x * rl, acc[e].y + v[e].y * rl);
    }
  }
#pragma unroll
  for (int e = 0; e < LS::E; ++e) {
    const int kz = LS::idxB(t, e);
    const R a = ssz[kz] * fx0, b = scz[kz] * fx1, c = scz[kz] * fx2;
    const R r2 = a * a + b * b + c * c;
    const R f = (r2 > R(0)) ? scale / r2 : R(0);
    acc[e] = cscale(acc[e], f);
  }
#pragma unroll 1
  for (int j = 0; j < 3; ++j) {
    C v[LS::E];
#pragma unroll
    for (int e = 0; e < LS::E; ++e) {
      const int kz = LS::idxB(t, e);
      const R rj = (j == 0) ? ssz[kz] * fx0 : scz[kz] * (j == 1 ? fx1 : fx2);
      v[e] = cscale(acc[e], rj);
    }
    LS::inv(v, lds + col, B, t, stw);
    if (kx != 0) {
      C* dst = base + (3 * i + j) * comp;
#pragma unroll
      for (int e = 0; e < LS::E; ++e) dst[LS::idxA(t, e) * plane] = v[e];
    }
  }
}

}  // namespace fg
