// Helpers of the kernels that hold whole transforms in registers.
#pragma once
#include "common.hpp"

namespace psfd {

// Buffer access of a complex value at a scalar plus a per-lane byte offset from a
// base that every lane holds alike: no lane keeps an address per element. (With
// plain pointers the compiler holds a 64-bit address per element from the loads
// to the stores.) Accesses beyond `bytes` read zero and store nothing.
struct LaneBuf {
  __amdgpu_buffer_rsrc_t r;
  PSFD_D LaneBuf(const void* p, unsigned bytes) {
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    r = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((unsigned long long)hi << 32) | lo), 0, bytes, 0x00020000);
  }
  PSFD_D void load(float2& x, unsigned lane, unsigned uni) const {
    const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, lane, uni, 0);
    x = make_float2(__uint_as_float(u[0]), __uint_as_float(u[1]));
  }
  // nontemporal: the line is not kept for a later reader
  PSFD_D void load_nt(float2& x, unsigned lane, unsigned uni) const {
    const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, lane, uni, 2);
    x = make_float2(__uint_as_float(u[0]), __uint_as_float(u[1]));
  }
  PSFD_D void load(double2& x, unsigned lane, unsigned uni) const {
    const auto u = __builtin_amdgcn_raw_buffer_load_b128(r, lane, uni, 0);
    x.x = __hiloint2double((int)u[1], (int)u[0]);
    x.y = __hiloint2double((int)u[3], (int)u[2]);
  }
  PSFD_D void store(float2 x, unsigned lane, unsigned uni) const {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    const u2 u = {__float_as_uint(x.x), __float_as_uint(x.y)};
    __builtin_amdgcn_raw_buffer_store_b64(u, r, lane, uni, 0);
  }
  PSFD_D void store(double2 x, unsigned lane, unsigned uni) const {
    typedef unsigned u4 __attribute__((ext_vector_type(4)));
    const u4 u = {(unsigned)__double2loint(x.x), (unsigned)__double2hiint(x.x), (unsigned)__double2loint(x.y),
                  (unsigned)__double2hiint(x.y)};
    __builtin_amdgcn_raw_buffer_store_b128(u, r, lane, uni, 0);
  }
};

// The value is formed here: without it the compiler sinks a finished transform
// behind the next barriers and branches, holding its inputs and twiddles instead.
PSFD_D void pin(float2& x) { asm volatile("" : "+v"(x.x), "+v"(x.y)); }
PSFD_D void pin(double2& x) { asm volatile("" : "+v"(x.x), "+v"(x.y)); }

}  // namespace psfd
