// Shared host/device helpers of the METok HIP library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <type_traits>

#include "device_once.h"
#include "metok.h"

namespace metok {

// ---------------------------------------------------------------------------------------------
// error reporting
// ---------------------------------------------------------------------------------------------
char* error_buffer();                       // thread-local, 512 bytes
int fail(int code, const char* fmt, ...);   // formats into the buffer, returns code
int check_launch(const char* what);         // hipGetLastError -> METOK_ERR_DEVICE
void clear_error();

// Measurement hook (metok_trace_kernel): brackets the launches of one kernel family with the caller's events.
struct KernelTrace { int kernel; hipEvent_t begin, end; };
KernelTrace& kernel_trace();                // thread-local
struct TraceScope {
    hipStream_t st;
    bool armed;
    TraceScope(int kernel, hipStream_t stream) : st(stream) {
        const KernelTrace& t = kernel_trace();
        armed = t.kernel == kernel && t.begin != nullptr && t.end != nullptr;
        if (armed) (void)hipEventRecord(t.begin, st);
    }
    ~TraceScope() { if (armed) (void)hipEventRecord(kernel_trace().end, st); }
};

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline size_t dtype_size(int dtype) { return dtype == METOK_BF16 ? 2 : 4; }
int ceil_ratio(double x);                   // ceil(x - 1e-9)

// Lets a kernel have `bytes` of dynamic LDS (the same for each of its launches): beyond 64 KB by an attribute of the current device's copy of it.
template <auto KERNEL>
bool allow_lds(size_t bytes) {
    if (bytes <= 64 * 1024) return true;
    static std::atomic<uint64_t> allowed{0};
    int device = 0;
    const bool ok = hipGetDevice(&device) == hipSuccess && once_per_device(allowed, device, [&] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)) == hipSuccess;
    });
    if (!ok) (void)hipGetLastError();       // the caller takes another kernel or reports the failure itself
    return ok;
}

constexpr int kWave = 64;

// ---------------------------------------------------------------------------------------------
// in-place row mover (stage3.hip): row i of a slab receives row idx[i] >= i.  Used by the KV
// compaction and by metok_prefill_prune when its output aliases its input.
// ---------------------------------------------------------------------------------------------
constexpr int kMaxLayersPerLaunch = 40;

struct RowMoveLayer {
    char* k;             // [B, Hkv, S_cap, row_bytes]
    char* v;             // second buffer of the layer (n_which == 2), else unused
    const int32_t* idx;  // [B, n_keep]
    int32_t n_keep;
    int32_t first_item;  // filled by launch_row_moves
    int32_t tiles;       // filled by launch_row_moves
    int32_t flag_slot;   // filled by launch_row_moves
    int32_t layer_id;    // index of the layer in per-layer tables (relink variant)
};

struct PlanArgs;                     // arguments of the planning kernel of the relink variant
struct RelinkTables {
    int64_t table_in_layer_stride;   // 0: one input table shared by the layers
    const int32_t* table_out;        // [L, B, pages_per_seq]
    const int32_t* home_page;        // [L, B, pages_per_seq]
    PlanArgs* plan;                  // launch_row_moves fills in the mover's geometry and launches the planning kernel
};

struct RowMoveGeom { int parts, lanes_per_row, rows_per_step, rows_per_tile; };

struct LengthTable { int n; int32_t len[METOK_MAX_LAYERS]; };

RowMoveGeom row_move_geom(int64_t row_bytes);
size_t row_move_workspace_bytes(int L, int B, int Hkv, int n_which, int64_t S_cap, int64_t row_bytes);
int launch_row_moves(RowMoveLayer* layers, int n_active, int B, int Hkv, int n_which, int64_t S_cap, int64_t row_bytes,
                     const int32_t* page_table, int page_size, int pages_per_seq, int64_t n_pages_pool,
                     int32_t* new_len, const int32_t* host_len, int L_total,
                     void* workspace, size_t workspace_bytes, hipStream_t st, const RelinkTables* relink);

// ---------------------------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------------------------
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2_t;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));   // 16 bytes, accepted by the non-temporal builtins

struct bf16_t { uint16_t bits; };           // storage type of a bf16 element

__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// Two fp32 values -> packed bf16 pair, round to nearest even: gfx950 converts a pair with one instruction.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2v_t __attribute__((ext_vector_type(2)));
    const f32x2_t v = {lo, hi};
    const bf16x2v_t r = __builtin_convertvector(v, bf16x2v_t);
    return __builtin_bit_cast(uint32_t, r);
}

// Streaming 16-byte load / store (non-temporal): on MI355X a copy of 0.15 to 0.8 GB runs at 6.7 TB/s with this hint and at 6.25
// without it, a pass that reads 0.6 to 1.7 GB 8 to 10 % faster; a read of 0.3 GB that was read just before gains nothing.
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream(uint4* p, const uint4& v) {
    const u32x4_t t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
}

// acc += a.lo * b.lo + a.hi * b.hi on two packed bf16 pairs, fp32 accumulate.
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc, false);
}

// 16-byte chunk arithmetic for the two element types.
template <typename T> struct Elem;
template <> struct Elem<bf16_t> {
    static constexpr int kVec = 8;
    static __device__ __forceinline__ float dot(const uint4& a, const uint4& b, float acc) {
        acc = dot2_bf16(a.x, b.x, acc);
        acc = dot2_bf16(a.y, b.y, acc);
        acc = dot2_bf16(a.z, b.z, acc);
        acc = dot2_bf16(a.w, b.w, acc);
        return acc;
    }
    static __device__ __forceinline__ void accumulate(const uint4& a, float (&acc)[8]) {
        acc[0] += bf16_lo(a.x); acc[1] += bf16_hi(a.x);
        acc[2] += bf16_lo(a.y); acc[3] += bf16_hi(a.y);
        acc[4] += bf16_lo(a.z); acc[5] += bf16_hi(a.z);
        acc[6] += bf16_lo(a.w); acc[7] += bf16_hi(a.w);
    }
};
template <> struct Elem<float> {
    static constexpr int kVec = 4;
    static __device__ __forceinline__ float dot(const uint4& a, const uint4& b, float acc) {
        acc = fmaf(__uint_as_float(a.x), __uint_as_float(b.x), acc);
        acc = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), acc);
        acc = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), acc);
        acc = fmaf(__uint_as_float(a.w), __uint_as_float(b.w), acc);
        return acc;
    }
    static __device__ __forceinline__ void accumulate(const uint4& a, float (&acc)[8]) {
        acc[0] += __uint_as_float(a.x); acc[1] += __uint_as_float(a.y);
        acc[2] += __uint_as_float(a.z); acc[3] += __uint_as_float(a.w);
    }
};

// Order-preserving map from float to uint32: a < b  <=>  key(a) < key(b) (-0 == +0, NaNs at the ends).  Keys run from 1 to
// 0xffffffff, so the difference of two keys is never 0xffffffff.
__device__ __forceinline__ uint32_t ordered_key(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? 0u - u : (u | 0x80000000u);      // -0 negates to the key of +0
}
__device__ __forceinline__ float score_of_key(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : 0u - key); }

// Sum over the 16 lanes of a DPP row; every lane of the row receives the total.
__device__ __forceinline__ float row16_sum(float v) {
    // row_ror:n rotates within each group of 16 lanes (dpp_ctrl 0x120 + n)
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x128, 0xf, 0xf, false));
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x124, 0xf, 0xf, false));
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x122, 0xf, 0xf, false));
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x121, 0xf, 0xf, false));
    return v;
}
// low half of the wave: a summed over the lane pairs (l, l + 32); high half: b likewise
__device__ __forceinline__ float swap32_add(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// even 16-lane rows: a of the rows (r, r + 1) added; odd rows: b likewise
__device__ __forceinline__ float swap16_add(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sum over all 64 lanes of the wave; every lane receives the total.
__device__ __forceinline__ float wave_sum(float v) {
    v = row16_sum(v);
    v = swap16_add(v, v);
    return swap32_add(v, v);
}
template <int G> __device__ __forceinline__ float group_sum(float v) {
    static_assert(G == 16 || G == 64, "token groups are one DPP row or one wave");
    return G == 16 ? row16_sum(v) : wave_sum(v);
}

// A batch of videos runs as one launch with blockIdx.z = video.  Pointer of that video, `bytes` (or `elems`
// elements) apart from its neighbours; NULL stays NULL.  A launch without a batch has blockIdx.z = 0.
template <typename P> __device__ __forceinline__ P* of_video(P* p, int64_t bytes) {
    using B = typename std::conditional<std::is_const<P>::value, const char, char>::type;
    return p ? reinterpret_cast<P*>(reinterpret_cast<B*>(p) + static_cast<int64_t>(blockIdx.z) * bytes) : p;
}
template <typename P> __device__ __forceinline__ P* of_video_elems(P* p, int64_t elems) {
    return p ? p + static_cast<int64_t>(blockIdx.z) * elems : p;
}

// A barrier that orders LDS accesses alone.  __syncthreads() also waits until this thread's global stores have completed,
// about 0.3 us each time in a workgroup that writes results between its steps.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP adds: shifts by 1, 2, 4, 8 inside the 16-lane rows, then the last
// lane of a row (of a pair of rows) is broadcast into the next one.  Every lane must be active.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ int dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int row16_inclusive_scan(int v) {
    v = dpp_add<0x111, 0xf>(v); v = dpp_add<0x112, 0xf>(v); v = dpp_add<0x114, 0xf>(v);
    return dpp_add<0x118, 0xf>(v);
}
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    v = row16_inclusive_scan(v);
    v = dpp_add<0x142, 0xa>(v);            // row_bcast:15 into rows 1 and 3
    return dpp_add<0x143, 0xc>(v);         // row_bcast:31 into rows 2 and 3
}

// Smallest / largest value of the 64 lanes of a wave; every lane receives it.  Every lane must be active.
template <bool MAX> __device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
    auto pick = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : (a < b ? a : b); };
    v = pick(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x128, 0xf, 0xf, false)));      // row_ror 8, 4, 2, 1
    v = pick(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x124, 0xf, 0xf, false)));
    v = pick(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x122, 0xf, 0xf, false)));
    v = pick(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x121, 0xf, 0xf, false)));
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = pick(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return pick(b[0], b[1]);
}

// Exclusive prefix sum of one int per thread over a workgroup of up to 1024 threads (whole waves); *total receives the sum.
// `scratch` is 16 ints of LDS that nobody reads any more; every wave scans the waves' totals for itself, so that one
// barrier is enough (a serial walk by one thread behind two barriers took 0.8 us).
__device__ __forceinline__ int block_exclusive_scan_lds(int v, int* scratch, int* total) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = (blockDim.x + 63) >> 6;
    const int incl = wave_inclusive_scan(v);
    if (lane == 63) scratch[wave] = incl;
    lds_barrier();
    const int sums = row16_inclusive_scan((lane & 15) < nwaves ? scratch[lane & 15] : 0);
    *total = __builtin_amdgcn_readlane(sums, 15);
    return (wave > 0 ? __builtin_amdgcn_readlane(sums, wave - 1) : 0) + incl - v;
}
// The same with 17 ints of LDS that may still be read from the call before, and with barriers that publish global stores too.
__device__ __forceinline__ int block_exclusive_scan(int v, int* scratch, int* total) {
    __syncthreads();
    return block_exclusive_scan_lds(v, scratch, total);
}

}  // namespace metok
