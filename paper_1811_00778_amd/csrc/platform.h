// Launch and memory shims.
//
// Every kernel of this library is written as a struct with
//   kThreads                      threads per workgroup
//   kPhases                       number of barrier-separated phases
//   struct Regs                   per-thread state that lives across barriers
//   template<int PH> phase(args, block, tid, lds, regs)
// and, optionally, a repeated prefix:
//   kLoopPhases, loop_count(args) phases [0, kLoopPhases) run loop_count times (Regs::iter = the iteration, a
//                                 barrier after every one of them), then the remaining phases once
// The HIP build runs the phases of one workgroup inside one __global__ function
// with __syncthreads() between phases.  The HCNN_HOSTEMU build (used only by the
// CPU test-suite to check kernel indexing and arithmetic before anything touches
// a GPU) runs the same phase bodies as plain loops over blocks and threads; it is
// a checker for the kernel sources, not a product path, and the Python binding
// never loads it.
// Optional: wave_sync(ph)       true: up to the next barrier the phases after ph touch only LDS words that no other
//                               wave touches in between, and no barrier stands after ph (of the last repeated phase: in front
//                               of what follows it, the next iteration or the rest).  The checker runs the phases
//                               between two barriers wave after wave, so that a wave which relies on another one is seen.
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <atomic>
#include <cstring>
#include <type_traits>
#include <utility>
#include <vector>

#ifdef HCNN_HOSTEMU
#define HCNN_HD inline
#define HCNN_HOSTDEV inline
#define HCNN_DEVICE_CODE 0
typedef int hcnn_hip_error_t;
typedef void* hcnn_stream_t;
#else
#include <hip/hip_runtime.h>
#define HCNN_HD __device__ __forceinline__
#define HCNN_HOSTDEV __host__ __device__ inline
typedef hipError_t hcnn_hip_error_t;
typedef hipStream_t hcnn_stream_t;
#endif

namespace hcnn {

#ifdef HCNN_HOSTEMU
struct alignas(16) U4 { uint32_t x, y, z, w; };
#else
typedef uint4 U4;
#endif

// opaque(x): x again, but as a value the compiler cannot trace back.  Used inside the repeated phases of a looped
// kernel on the thread index, so that the per-thread addresses derived from it are recomputed in every iteration
// (a few instructions) rather than computed once, kept across the whole loop and spilled.
HCNN_HD int opaque(int x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
  return x;
}

// ldc(table, i): element i of a read-only table (moduli, twiddles, base-conversion constants).
// In device code the words are read through the constant address space: with a wave-uniform
// index the compiler then issues scalar loads instead of one vector load per lane.  The tables
// are written once, before any kernel runs, and never by a kernel.
#if defined(__HIP_DEVICE_COMPILE__)
template <class T>
__device__ __forceinline__ T ldc(const T* table, size_t i) {
  static_assert(sizeof(T) % 4 == 0 && alignof(T) >= 4, "tables are made of 32-bit words");
  typedef const uint32_t __attribute__((address_space(4))) * cptr;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
  cptr w = (cptr)(table + i);
#pragma clang diagnostic pop
  T out;
  uint32_t* o = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
  for (unsigned k = 0; k < sizeof(T) / 4; ++k) o[k] = w[k];
  return out;
}
#elif defined(HCNN_HOSTEMU)
template <class T> inline T ldc(const T* table, size_t i) { return table[i]; }
#else
template <class T> __device__ __forceinline__ T ldc(const T* table, size_t i) { return table[i]; }
#endif

// Accesses of the form uniform base + 32-bit byte offset per lane.  On the device the base is pinned to scalar registers,
// so that the access takes it as it is: written as an array index, the compiler moves compile-time parts of the offset
// behind the per-lane part and spends a 64-bit vector addition on every access.
// ldc_at: from a read-only table, by scalar loads where the offset is wave-uniform.
#if defined(__HIP_DEVICE_COMPILE__)
typedef uint32_t hcnn_word4 __attribute__((ext_vector_type(4)));
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wold-style-cast"
template <class T>
__device__ __forceinline__ T ldc_at(const T* table, uint32_t byte_off) {
  static_assert(sizeof(T) == 4 || (sizeof(T) == 16 && alignof(T) == 16), "one word or one aligned 16-byte word");
  typedef std::conditional_t<sizeof(T) == 4, uint32_t, hcnn_word4> word;
  typedef const word __attribute__((address_space(4))) * cptr;
  typedef const char __attribute__((address_space(4))) * bptr;
  return __builtin_bit_cast(T, *(cptr)((bptr)table + byte_off));
}
__device__ __forceinline__ uint32_t ld_at(const uint32_t* base, uint32_t byte_off) {
  typedef const uint32_t __attribute__((address_space(1))) * gptr;
  typedef const char __attribute__((address_space(1))) * bptr;
  bptr b = (bptr)base;
  asm("" : "+s"(b));
  return *(gptr)(b + byte_off);
}
__device__ __forceinline__ U4 ld4_at(const uint32_t* base, uint32_t byte_off) {
  typedef const hcnn_word4 __attribute__((address_space(1))) * gptr;
  typedef const char __attribute__((address_space(1))) * bptr;
  bptr b = (bptr)base;
  asm("" : "+s"(b));
  const hcnn_word4 w = *(gptr)(b + byte_off);
  U4 r; r.x = w.x; r.y = w.y; r.z = w.z; r.w = w.w;
  return r;
}
__device__ __forceinline__ void st_at(uint32_t* base, uint32_t byte_off, uint32_t v) {
  typedef uint32_t __attribute__((address_space(1))) * gptr;
  typedef char __attribute__((address_space(1))) * bptr;
  bptr b = (bptr)base;
  asm("" : "+s"(b));
  *(gptr)(b + byte_off) = v;
}
__device__ __forceinline__ void st4_at(uint32_t* base, uint32_t byte_off, U4 v) {
  typedef hcnn_word4 __attribute__((address_space(1))) * gptr;
  typedef char __attribute__((address_space(1))) * bptr;
  bptr b = (bptr)base;
  asm("" : "+s"(b));
  *(gptr)(b + byte_off) = hcnn_word4{v.x, v.y, v.z, v.w};
}
#pragma clang diagnostic pop
#else
template <class T> HCNN_HD T ldc_at(const T* table, uint32_t byte_off) { return table[byte_off / sizeof(T)]; }
HCNN_HD uint32_t ld_at(const uint32_t* base, uint32_t byte_off) { return base[byte_off / 4]; }
HCNN_HD U4 ld4_at(const uint32_t* base, uint32_t byte_off) { return *reinterpret_cast<const U4*>(base + byte_off / 4); }
HCNN_HD void st_at(uint32_t* base, uint32_t byte_off, uint32_t v) { base[byte_off / 4] = v; }
HCNN_HD void st4_at(uint32_t* base, uint32_t byte_off, U4 v) { *reinterpret_cast<U4*>(base + byte_off / 4) = v; }
#endif

// Division of a workgroup index by a launch constant: m = floor(2^32 / d), or 2^32 - 1 for d = 1 (the estimate is the
// quotient or one less).  (A run-time divisor otherwise costs a floating-point reciprocal and its corrections in every phase.)
struct FastDiv { uint32_t d, m; };
inline FastDiv fast_div(uint32_t d) { return FastDiv{d, d == 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / d)}; }
HCNN_HD uint32_t quot(uint32_t x, FastDiv f) {
#if defined(HCNN_HOSTEMU)
  const uint32_t q = (uint32_t)(((uint64_t)x * f.m) >> 32);
#else
  const uint32_t q = __umulhi(x, f.m);
#endif
  return x - q * f.d >= f.d ? q + 1 : q;
}

// The value as it is, but not one the compiler can trace back to where it came from.
template <class T>
HCNN_HD T untraced(T x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("" : "+v"(x));
#endif
  return x;
}

// No instruction is scheduled across this point (loads in front of it are issued before what follows)
HCNN_HD void sched_fence() {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}

// x, known to be the same in all lanes of a wave, as a scalar
HCNN_HD uint32_t wave_uniform(uint32_t x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
#else
  return x;
#endif
}

// kMinWavesPerSimd (optional): occupancy the register allocation of the kernel must allow
template <class K, class = void> struct MinWavesPerSimd { static constexpr int value = 1; };
template <class K> struct MinWavesPerSimd<K, std::void_t<decltype(K::kMinWavesPerSimd)>> { static constexpr int value = K::kMinWavesPerSimd; };
template <class K, class = void> struct WaveSync { static constexpr bool after(int) { return false; } };
template <class K> struct WaveSync<K, std::void_t<decltype(K::wave_sync(0))>> { static constexpr bool after(int ph) { return K::wave_sync(ph); } };
template <class K, class = void> struct LoopPhases { static constexpr int value = 0; };
template <class K> struct LoopPhases<K, std::void_t<decltype(K::kLoopPhases)>> { static constexpr int value = K::kLoopPhases; };

#ifdef HCNN_HOSTEMU
// ------------------------------------------------------------------ host emulation
// What a test may set (hcnn_emu_device): compute units of the contexts created from then on, the largest allocation that is granted
static uint32_t emu_units = 1;           // small rounds: the checker's little batches reach every batch-splitting path
static size_t emu_largest = ~(size_t)0;
inline int dev_malloc(void** p, size_t bytes) {
  *p = bytes <= emu_largest ? std::malloc(bytes ? bytes : 1) : nullptr;
  return *p ? 0 : 2;
}
inline int dev_free(void* p) { std::free(p); return 0; }
inline int dev_memset(void* p, int v, size_t bytes, hcnn_stream_t) { std::memset(p, v, bytes); return 0; }
inline int copy_h2d(void* d, const void* h, size_t bytes, hcnn_stream_t) { std::memcpy(d, h, bytes); return 0; }
inline int copy_d2h(void* h, const void* d, size_t bytes, hcnn_stream_t) { std::memcpy(h, d, bytes); return 0; }
inline int copy_d2d(void* d, const void* s, size_t bytes, hcnn_stream_t) { std::memmove(d, s, bytes); return 0; }
inline int stream_sync(hcnn_stream_t) { return 0; }
typedef int hcnn_event_t;
inline int event_create(hcnn_event_t* e) { *e = 0; return 0; }
inline int event_destroy(hcnn_event_t) { return 0; }
inline int event_record(hcnn_event_t, hcnn_stream_t) { return 0; }
inline int event_elapsed_ms(float* ms, hcnn_event_t, hcnn_event_t) { *ms = 0.f; return 0; }
inline size_t max_lds_bytes() { return 160 * 1024; }
inline uint32_t compute_unit_count() { return emu_units; }
HCNN_HD void atomic_inc64(unsigned long long* p) { *p += 1; }
HCNN_HD void atomic_max32(uint32_t* p, uint32_t v) { if (v > *p) *p = v; }
// on LDS words, returning the value before
HCNN_HD uint32_t lds_or(uint32_t* p, uint32_t v) { const uint32_t o = *p; *p = o | v; return o; }
HCNN_HD uint32_t lds_add(uint32_t* p, uint32_t v) { const uint32_t o = *p; *p = o + v; return o; }
// Workgroups of kernel K that one compute unit holds at a time.  The checker has no device to ask: it counts 16
// wavefronts per compute unit (8 for workgroups of 256 threads, the shape whose register use halves the occupancy
// on the device), which with its single compute unit gives rounds of a few workgroups.
template <class K, class Args>
int resident_workgroups_per_cu(size_t, int* out) {
  const int waves = K::kThreads / 64 > 0 ? K::kThreads / 64 : 1;
  *out = (K::kThreads == 256 ? 8 : 16) / waves;
  if (*out < 1) *out = 1;
  return 0;
}

template <class K, class Args>
using EmuPhase = void (*)(const Args&, unsigned, int, uint32_t*, typename K::Regs&);
template <class K, class Args, int... PH>
EmuPhase<K, Args> emu_phase(int ph, std::integer_sequence<int, PH...>) {
  static constexpr EmuPhase<K, Args> all[] = {[](const Args& a, unsigned bid, int tid, uint32_t* lds, typename K::Regs& r) {
    K::template phase<PH>(a, bid, tid, lds, r);
  }...};
  return all[ph];
}

template <class K, class Args>
int launch(hcnn_stream_t, size_t grid, size_t lds_bytes, const Args& a) {
  if (lds_bytes > max_lds_bytes()) return 1;
  std::vector<uint32_t> lds(lds_bytes / 4 + 4);
  std::vector<typename K::Regs> regs(K::kThreads);
  constexpr int LP = LoopPhases<K>::value;
  // the phases of a workgroup in order; `next`: the first one behind the next barrier
  struct Step { EmuPhase<K, Args> run; uint32_t iter; size_t next; };
  std::vector<Step> steps;
  std::vector<bool> barrier;
  auto add = [&](int ph, uint32_t it) {
    steps.push_back(Step{emu_phase<K, Args>(ph, std::make_integer_sequence<int, K::kPhases>{}), it, 0});
    barrier.push_back(!WaveSync<K>::after(ph));
  };
  uint32_t count = 0;
  if constexpr (LP > 0) {
    count = K::loop_count(a);
    for (uint32_t it = 0; it < count; ++it)
      for (int ph = 0; ph < LP; ++ph) add(ph, it);
  }
  for (int ph = LP; ph < K::kPhases; ++ph) add(ph, count);
  for (size_t i = steps.size(); i-- > 0;) steps[i].next = i + 1 == steps.size() || barrier[i] ? i + 1 : steps[i + 1].next;
  const int waves = (K::kThreads + 63) / 64;
  for (size_t bid = 0; bid < grid; ++bid) {
    bool up = true;                                    // waves in ascending, then in descending order
    for (size_t s = 0; s < steps.size(); s = steps[s].next, up = !up)
      for (int w = 0; w < waves; ++w)
        for (size_t i = s; i < steps[s].next; ++i) {
          const int t0 = (up ? w : waves - 1 - w) * 64, t1 = t0 + 64 < K::kThreads ? t0 + 64 : K::kThreads;
          for (int tid = t0; tid < t1; ++tid) {
            if constexpr (LP > 0) regs[tid].iter = steps[i].iter;
            steps[i].run(a, (unsigned)bid, tid, lds.data(), regs[tid]);
          }
        }
  }
  return 0;
}

#else
// ------------------------------------------------------------------ HIP
inline int dev_malloc(void** p, size_t bytes) {
  const hipError_t e = hipMalloc(p, bytes ? bytes : 1);
  if (e != hipSuccess) (void)hipGetLastError();      // reported here, not by the next launch
  return (int)e;
}
inline int dev_free(void* p) { return (int)hipFree(p); }
inline int dev_memset(void* p, int v, size_t bytes, hcnn_stream_t s) { return (int)hipMemsetAsync(p, v, bytes, s); }
inline int copy_h2d(void* d, const void* h, size_t bytes, hcnn_stream_t s) {
  // tables are tiny and built once: a synchronous copy keeps the host vector's lifetime simple
  (void)s;
  return (int)hipMemcpy(d, h, bytes, hipMemcpyHostToDevice);
}
inline int copy_d2h(void* h, const void* d, size_t bytes, hcnn_stream_t s) {
  int e = (int)hipStreamSynchronize(s);
  if (e) return e;
  return (int)hipMemcpy(h, d, bytes, hipMemcpyDeviceToHost);
}
inline int copy_d2d(void* d, const void* s_, size_t bytes, hcnn_stream_t s) {
  return (int)hipMemcpyAsync(d, s_, bytes, hipMemcpyDeviceToDevice, s);
}
inline int stream_sync(hcnn_stream_t s) { return (int)hipStreamSynchronize(s); }
typedef hipEvent_t hcnn_event_t;
inline int event_create(hcnn_event_t* e) { return (int)hipEventCreate(e); }
inline int event_destroy(hcnn_event_t e) { return (int)hipEventDestroy(e); }
inline int event_record(hcnn_event_t e, hcnn_stream_t s) { return (int)hipEventRecord(e, s); }
inline int event_elapsed_ms(float* ms, hcnn_event_t a, hcnn_event_t b) { return (int)hipEventElapsedTime(ms, a, b); }
inline size_t max_lds_bytes() {
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return 0;
  return (size_t)v;
}
inline uint32_t compute_unit_count() {
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) return 256;
  return (uint32_t)v;
}
HCNN_HD void atomic_inc64(unsigned long long* p) { atomicAdd(p, 1ull); }
HCNN_HD void atomic_max32(uint32_t* p, uint32_t v) { atomicMax(p, v); }
HCNN_HD uint32_t lds_or(uint32_t* p, uint32_t v) { return atomicOr(p, v); }
HCNN_HD uint32_t lds_add(uint32_t* p, uint32_t v) { return atomicAdd(p, v); }

// What separates phase PH from the next one.  A wave's own LDS accesses take effect in order, so that between phases that
// exchange data within a wave only the compiler has to be kept from reordering them.
template <class K, int PH>
__device__ __forceinline__ void phase_sync() {
  if constexpr (WaveSync<K>::after(PH)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

template <class K, int PH, int END, class Args>
__device__ __forceinline__ void run_phases(const Args& a, unsigned bid, int tid, uint32_t* lds,
                                           typename K::Regs& regs) {
  K::template phase<PH>(a, bid, tid, lds, regs);
  if constexpr (PH + 1 < END) {
    phase_sync<K, PH>();
    run_phases<K, PH + 1, END, Args>(a, bid, tid, lds, regs);
  }
}

template <class K, class Args>
__global__ void __launch_bounds__(K::kThreads, MinWavesPerSimd<K>::value) kernel_entry(const Args a) {
  extern __shared__ __align__(16) uint32_t hcnn_lds[];
  typename K::Regs regs;
  constexpr int LP = LoopPhases<K>::value;
  if constexpr (LP > 0) {
    const uint32_t count = K::loop_count(a);
    for (uint32_t it = 0; it < count; ++it) {
      regs.iter = it;
      run_phases<K, 0, LP, Args>(a, blockIdx.x, (int)threadIdx.x, hcnn_lds, regs);
      phase_sync<K, LP - 1>();
    }
    regs.iter = count;
  }
  if constexpr (LP < K::kPhases) run_phases<K, LP, K::kPhases, Args>(a, blockIdx.x, (int)threadIdx.x, hcnn_lds, regs);
}

template <class K, class Args>
int launch(hcnn_stream_t s, size_t grid, size_t lds_bytes, const Args& a) {
  if (grid == 0) return 0;
  if (grid > 0x7fffffffull) return (int)hipErrorInvalidConfiguration;
  if (lds_bytes > 48 * 1024) {
    // raised once per kernel and size (not on every launch, and so not while a caller records a graph after its
    // warm-up call)
    static std::atomic<size_t> allowed{0};
    if (lds_bytes > allowed.load(std::memory_order_relaxed)) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&kernel_entry<K, Args>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
      if (e != hipSuccess) return (int)e;
      allowed.store(lds_bytes, std::memory_order_relaxed);
    }
  }
  hipLaunchKernelGGL((kernel_entry<K, Args>), dim3((unsigned)grid), dim3(K::kThreads), lds_bytes, s, a);
  return (int)hipGetLastError();
}

// Workgroups of kernel K (with lds_bytes of dynamic LDS each) that one compute unit holds at a time, as the runtime
// derives it from the compiled kernel's register and LDS use.
template <class K, class Args>
int resident_workgroups_per_cu(size_t lds_bytes, int* out) {
  if (lds_bytes > 48 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&kernel_entry<K, Args>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return (int)e;
  }
  int n = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel_entry<K, Args>, K::kThreads, lds_bytes);
  if (e != hipSuccess) return (int)e;
  *out = n > 0 ? n : 1;
  return 0;
}
#endif

}  // namespace hcnn
