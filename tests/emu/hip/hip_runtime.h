// A CPU stand-in for the HIP headers: enough of the language to compile the
// library's one-block device code as C++ and run a block of it work-item by
// work-item (block_emu.cpp).  Work-items of a wavefront run one after another
// between the operations that join them, block barriers included.
#pragma once
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstring>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline
#define __noinline__
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) alignas(n)

struct alignas(16) double2 { double x, y; };
struct alignas(8) float2 { float x, y; };
struct dim3 { unsigned x, y, z; dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {} };
typedef struct emu_stream *hipStream_t;
typedef struct emu_event *hipEvent_t;
typedef int hipError_t;
using std::isfinite;

namespace emu {
extern dim3 thread_idx, block_idx, block_dim, grid_dim;   // of the running work-item
void barrier(const char *file, int line);
// every live lane of the wavefront hands in a word; the words of all 64 (0 of a lane that has ended)
const unsigned long long *exchange(unsigned long long word);
struct Pair { unsigned v[2]; unsigned operator[](int i) const { return v[i]; } };
inline int lane() { return thread_idx.x & 63; }
inline Pair swap(unsigned a, unsigned b, int w) {
    const unsigned long long *x = exchange((unsigned long long)b << 32 | a);
    const int i = lane();
    Pair p;
    p.v[0] = (i & w) ? (unsigned)(x[i - w] >> 32) : (unsigned)x[i];
    p.v[1] = (i & w) ? (unsigned)(x[i] >> 32) : (unsigned)x[i + w];
    return p;
}
// the DPP forms the library uses: quad permute, row shift left/right, row rotate right
inline int dpp(int old, int src, int ctrl, int bank_mask) {
    const unsigned long long *x = exchange((unsigned)src);
    const int i = lane(), r = i & 15, row = i & 48;
    if (!((bank_mask >> (r >> 2)) & 1)) return old;
    if (ctrl < 0x100) return (int)x[(i & 60) + ((ctrl >> (2 * (i & 3))) & 3)];
    const int n = ctrl & 15;
    if ((ctrl & 0xF0) == 0x20) return (int)x[row + ((r - n) & 15)];
    const int from = (ctrl & 0xF0) == 0x00 ? r + n : r - n;
    return from < 0 || from > 15 ? old : (int)x[row + from];
}
template <typename V> inline V shuffle(V v, int from) {
    unsigned long long w = 0;
    std::memcpy(&w, &v, sizeof(V));
    w = exchange(w)[from & 63];
    std::memcpy(&v, &w, sizeof(V));
    return v;
}
inline unsigned long long ballot(bool p) {
    const unsigned long long *x = exchange(p ? 1 : 0);
    unsigned long long m = 0;
    for (int i = 0; i < 64; ++i) m |= x[i] << i;
    return m;
}
inline unsigned brev(unsigned v) {
    unsigned r = 0;
    for (int i = 0; i < 32; ++i) r |= ((v >> i) & 1u) << (31 - i);
    return r;
}
inline int lo(double v) { unsigned long long w; std::memcpy(&w, &v, 8); return (int)(unsigned)w; }
inline int hi(double v) { unsigned long long w; std::memcpy(&w, &v, 8); return (int)(unsigned)(w >> 32); }
inline double join(int h, int l) {
    const unsigned long long w = (unsigned long long)(unsigned)h << 32 | (unsigned)l;
    double v;
    std::memcpy(&v, &w, 8);
    return v;
}
}  // namespace emu

#define threadIdx emu::thread_idx
#define blockIdx emu::block_idx
#define blockDim emu::block_dim
#define gridDim emu::grid_dim
#define __syncthreads() emu::barrier(__FILE__, __LINE__)
#define __builtin_amdgcn_permlane32_swap(a, b, c, d) emu::swap(a, b, 32)
#define __builtin_amdgcn_permlane16_swap(a, b, c, d) emu::swap(a, b, 16)
#define __builtin_amdgcn_update_dpp(old, src, ctrl, row, bank, bound) emu::dpp(old, src, ctrl, bank)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __shfl_xor(v, off, w) emu::shuffle(v, emu::lane() ^ (off))
#define __shfl_down(v, off, w) emu::shuffle(v, emu::lane() + (off) < 64 ? emu::lane() + (off) : emu::lane())
#define __ballot(p) emu::ballot(p)
#define __any(p) (emu::ballot(p) != 0)
#define __popcll(x) __builtin_popcountll(x)
#define __brev(x) emu::brev(x)
#define __double2loint(v) emu::lo(v)
#define __double2hiint(v) emu::hi(v)
#define __hiloint2double(h, l) emu::join(h, l)
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) ((void)0)
