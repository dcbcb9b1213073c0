// Pulls and node storage shared by the D3Q19 steps (kernels3d.hip, flat3d.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "devcase.hpp"

namespace vclb {

// Node offsets of one 3D pull: the writer of direction i sits at x - c_i, reached from
// the node's own index s0 by one of xm / xp, ym / yp, zm / zp per axis (the wrapped steps
// to x - 1 / x + 1 and so on; x and z are periodic).  With walls bounding y, lo / hi mark
// the first / last row, where the directions coming from behind the wall are the node's
// own opposite populations (half-way bounce-back).
struct Nbr3 {
  int s0, xm, xp, ym, yp, zm, zp;
  bool lo, hi;
};

__device__ __forceinline__ Nbr3 nbr3(int x, int y, int z, int nx, int ny, int nz, int nxy, bool wall) {
  Nbr3 o;
  o.s0 = x + nx * y + nxy * z;
  o.lo = wall && y == 0;
  o.hi = wall && y == ny - 1;
  o.xm = x == 0 ? nx - 1 : -1;
  o.xp = x == nx - 1 ? 1 - nx : 1;
  o.ym = y == 0 ? (ny - 1) * nx : -nx;
  o.yp = y == ny - 1 ? (1 - ny) * nx : nx;
  o.zm = z == 0 ? (nz - 1) * nxy : -nxy;
  o.zp = z == nz - 1 ? (1 - nz) * nxy : nxy;
  return o;
}

// Offset of the writer of direction i from the uniform base of its plane: the node's own
// index s0 moved by one of xm / xp, ym / yp, zm / zp per axis.
template <int i>
__device__ __forceinline__ int pull_index(const Nbr3& o) {
  using L = D3Q19;
  int s = o.s0;
  if constexpr (L::cx[i] > 0) s += o.xm;
  if constexpr (L::cx[i] < 0) s += o.xp;
  if constexpr (L::cy[i] > 0) s += o.ym;
  if constexpr (L::cy[i] < 0) s += o.yp;
  if constexpr (L::cz[i] > 0) s += o.zm;
  if constexpr (L::cz[i] < 0) s += o.zp;
  return s;
}

// Buffer-resource access, for periodic cases whose arrays each span less than 2 GiB: one
// resource per array (uniform), the plane's byte offset as the scalar offset (the same
// scalar for every array of equal plane stride) and the node's byte offset as the vector
// offset, so that an access needs one 32-bit offset per lane and no 64-bit address.
struct Bufs3 {
  __amdgpu_buffer_rsrc_t g, f, phis, gd, fd, phisd, J;   // read: g, f, phis; written: gd, fd, phisd; J both
  int pb;   // bytes per population plane (ns entries of the stored type)
  int jb;   // bytes per plane of J
};
// fourth word of a raw (unswizzled, unstrided) buffer resource on gfx9-family GPUs:
// 32-bit data format, every destination selector zero
constexpr int kRawBufferWord3 = 0x00020000;

template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const T* p, long entries) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), short(0), int(entries * long(sizeof(T))),
                                           kRawBufferWord3);
}
template <class T>
__device__ __forceinline__ T buf_ld(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff) {
  if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <class T>
__device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff, T v) {
  if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, voff, soff, 0);
  else {
    using U2 = unsigned __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, voff, soff, 0);
  }
}
// a population in the storage's form: decoded to / encoded from the arithmetic type
template <class St>
__device__ __forceinline__ typename St::R buf_load_pop(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff) {
  if constexpr (sizeof(typename St::S) == 2)
    return __half2float(__ushort_as_half(__builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0)));
  else return buf_ld<typename St::S>(r, voff, soff);
}
template <class St>
__device__ __forceinline__ void buf_store_pop(__amdgpu_buffer_rsrc_t r, unsigned voff, int soff,
                                              typename St::R v) {
  if constexpr (sizeof(typename St::S) == 2)
    __builtin_amdgcn_raw_buffer_store_b16(__half_as_ushort(__float2half_rn(v)), r, voff, soff, 0);
  else buf_st<typename St::S>(r, voff, soff, typename St::S(v));
}

// The 19 pulls at one node: 32-bit node offsets from the uniform base of each direction's
// plane (planes of ns entries; the case has fewer than 2^31 nodes), accessed with index type
// IX (unsigned: 32-bit byte offsets, when n times the element size fits them).  ps (shifted
// storage): the phi the stored deviations refer to, this node's own phis entry.
template <class St, class IX>
__device__ __forceinline__ void pull19_ptr(const typename St::S* __restrict__ src, const float* __restrict__ phis,
                                           long ns, const Nbr3& o, typename St::R (&out)[19], typename St::R* ps) {
  using L = D3Q19;
  using R = typename St::R;
  static_for<0, L::Q>([&](auto I) {
    constexpr int i = decltype(I)::value;
    int s = pull_index<i>(o);
    const typename St::S* base = src + i * ns;
    if constexpr (L::cy[i] > 0) {   // from the row below: behind the bottom wall at y = 0
      if (o.lo) {
        s = o.s0;
        base = src + L::opp[i] * ns;
      }
    }
    if constexpr (L::cy[i] < 0) {   // from the row above: behind the top wall at y = ny - 1
      if (o.hi) {
        s = o.s0;
        base = src + L::opp[i] * ns;
      }
    }
    out[i] = St::load(base, IX(s));
  });
  if constexpr (St::shifted) {   // every deviation refers to this node's own phis entry
    if (ps) {
      const R own = R(ldg(phis, IX(o.s0)));
#pragma unroll
      for (int i = 0; i < L::Q; ++i) ps[i] = own;
    }
  }
}

// The same by the kernel's form of access.  BUF: through the buffer resources rs (the set)
// and rph (phis), planes pb bytes apart; periodic cases only (no pull is redirected at a
// wall).
template <class St, class IX, bool BUF>
__device__ __forceinline__ void pull19(const typename St::S* __restrict__ src, const float* __restrict__ phis,
                                       long ns, __amdgpu_buffer_rsrc_t rs, __amdgpu_buffer_rsrc_t rph, int pb,
                                       const Nbr3& o, typename St::R (&out)[19], typename St::R* ps) {
  using L = D3Q19;
  using R = typename St::R;
  if constexpr (BUF) {
    static_for<0, L::Q>([&](auto I) {
      constexpr int i = decltype(I)::value;
      out[i] = buf_load_pop<St>(rs, unsigned(pull_index<i>(o)) * unsigned(sizeof(typename St::S)), i * pb);
    });
    if constexpr (St::shifted) {
      if (ps) {
        const R own = R(buf_ld<float>(rph, unsigned(o.s0) * 4u, 0));
#pragma unroll
        for (int i = 0; i < L::Q; ++i) ps[i] = own;
      }
    }
  } else {
    pull19_ptr<St, IX>(src, phis, ns, o, out, ps);
  }
}

// phi and psi of a node side by side: one 2-word LDS access per stencil point
template <class R>
struct alignas(2 * sizeof(R)) PhiPsi3 {
  R phi, psi;
};

}  // namespace vclb
