// Device helpers the sampler kernels share: wave reductions, the squared distance, and the words workgroups exchange.
#ifndef FASTPOINT_WAVE_H_
#define FASTPOINT_WAVE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#pragma clang fp contract(off)

namespace fastpoint {
namespace {

constexpr float kPadCoord = 3.0e38f;    // coordinates of slots beyond N: every distance becomes +inf
constexpr uint32_t kNoIdx = 0xFFFFFFFFu;

// ---------------------------------------------------------------- wave helpers
// Values that are equal in all lanes but come out of LDS or cross-lane operations: telling the
// compiler so keeps the control flow that depends on them on the scalar unit.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ uint32_t uni(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ float unif(float v)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}
__device__ __forceinline__ uint64_t uni64(uint64_t v)
{
    return ((uint64_t)uni((uint32_t)(v >> 32)) << 32) | (uint64_t)uni((uint32_t)v);
}
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v)
{
    // every lane has a valid source for the controls used here, so bound_ctrl is irrelevant;
    // this form lets the compiler fuse the move into the following min/max
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
// after these four steps every lane holds the reduction over its row of 16 lanes
__device__ __forceinline__ uint32_t row_max_u32(uint32_t v)
{
    v = max(v, dpp<0xB1>(v));    // quad_perm [1,0,3,2]
    v = max(v, dpp<0x4E>(v));    // quad_perm [2,3,0,1]
    v = max(v, dpp<0x141>(v));   // row_half_mirror
    v = max(v, dpp<0x140>(v));   // row_mirror
    return v;
}
__device__ __forceinline__ uint32_t row_min_u32(uint32_t v)
{
    v = min(v, dpp<0xB1>(v));
    v = min(v, dpp<0x4E>(v));
    v = min(v, dpp<0x141>(v));
    v = min(v, dpp<0x140>(v));
    return v;
}
__device__ __forceinline__ uint32_t rdlane(uint32_t v, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ float rdlane_f(float v, int l)
{
    return __uint_as_float(rdlane(__float_as_uint(v), l));
}
// puts a wave-uniform value into lane `lane` of v
__device__ __forceinline__ void set_lane(uint32_t& v, int my_lane, int lane, uint32_t uniform_value)
{
    v = my_lane == lane ? uniform_value : v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = row_max_u32(v);
    return max(max(rdlane(v, 0), rdlane(v, 16)), max(rdlane(v, 32), rdlane(v, 48)));     // scalar unit
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v)
{
    v = row_min_u32(v);
    return min(min(rdlane(v, 0), rdlane(v, 16)), min(rdlane(v, 32), rdlane(v, 48)));
}
// maximum over the wave as a scalar-unit value: the loop that uses it branches on it
__device__ __forceinline__ uint32_t smax(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("s_max_u32 %0, %1, %2" : "=s"(r) : "s"(a), "s"(b) : "scc");
    return r;
}
__device__ __forceinline__ uint32_t wave_max_scalar(uint32_t v)
{
    v = row_max_u32(v);
    return smax(smax(rdlane(v, 0), rdlane(v, 16)), smax(rdlane(v, 32), rdlane(v, 48)));
}
// inclusive prefix sum over the lanes of a wave: inside a row of 16 lanes by shifts of 1, 2, 4, 8
// (a lane whose source lies outside its row adds 0), then the totals of the rows in front
__device__ __forceinline__ int wave_incl_sum(int v, int lane)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);    // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);    // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);    // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);    // row_shr:8
    const int r0 = (int)rdlane((uint32_t)v, 15), r1 = (int)rdlane((uint32_t)v, 31), r2 = (int)rdlane((uint32_t)v, 47);
    const int row = lane >> 4;
    return v + (row > 0 ? r0 : 0) + (row > 1 ? r1 : 0) + (row > 2 ? r2 : 0);
}
__device__ __forceinline__ int first_lane(uint64_t mask) { return __builtin_ctzll(mask); }
__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// squared distance, ((dx*dx)+(dy*dy))+(dz*dz), each operation rounded on its own
__device__ __forceinline__ float dist2(float ax, float ay, float az, float bx, float by, float bz)
{
    float dx = ax - bx;
    float dy = ay - by;
    float dz = az - bz;
    float t = dx * dx;
    t = t + dy * dy;
    t = t + dz * dz;
    return t;
}

// ------------------------------------------------- words exchanged between workgroups
__device__ __forceinline__ void ll_store(uint64_t* p, uint32_t val, uint32_t stamp)
{
    __hip_atomic_store(p, ((uint64_t)stamp << 32) | (uint64_t)val, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ll_load(const uint64_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits until the NW words at p carry `stamp`; false if the wait limit expired.
template <int NWORDS>
__device__ __forceinline__ bool ll_wait(const uint64_t* p, uint32_t stamp, uint32_t (&val)[NWORDS],
                                        int64_t wait_ticks)
{
    int64_t t0 = 0;
    for (uint32_t spin = 0;; ++spin) {
        uint64_t v[NWORDS];
#pragma unroll
        for (int k = 0; k < NWORDS; ++k) v[k] = ll_load(p + k);
        bool ok = true;
#pragma unroll
        for (int k = 0; k < NWORDS; ++k) ok = ok && ((uint32_t)(v[k] >> 32) == stamp);
        if (ok) {
#pragma unroll
            for (int k = 0; k < NWORDS; ++k) val[k] = (uint32_t)v[k];
            return true;
        }
        if ((spin & 63u) == 63u || wait_ticks <= 0) {
            int64_t now = (int64_t)wall_clock64();
            if (t0 == 0) t0 = now;
            else if (now - t0 > wait_ticks) return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The same for one word, with four reads under way a sixth of a trip apart: a trip takes some 700 ns, and waiting for the
// answer before asking again finds the word half a trip late on average.
__device__ __forceinline__ bool ll_wait_close(const uint64_t* p, uint32_t stamp, uint32_t& val, int64_t wait_ticks)
{
    constexpr int N = 4;
    uint64_t v[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        v[k] = ll_load(p);
        if (k + 1 < N) __builtin_amdgcn_s_sleep(3);
    }
    int64_t t0 = 0;
    for (uint32_t spin = 0;; ++spin) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
            if ((uint32_t)(v[k] >> 32) == stamp) {
                val = (uint32_t)v[k];
                return true;
            }
            v[k] = ll_load(p);
        }
        if ((spin & 15u) == 15u || wait_ticks <= 0) {
            const int64_t now = (int64_t)wall_clock64();
            if (t0 == 0) t0 = now;
            else if (now - t0 > wait_ticks) return false;
        }
    }
}

struct Rec {          // one arg-max candidate: squared distance bits, index, coordinates
    uint32_t d, idx;
    float x, y, z;
    uint32_t fail;
    uint32_t pad0, pad1;
};

// reduce `nrec` records held by lanes 0..nrec-1 of a wave (nrec <= 64)
__device__ __forceinline__ Rec reduce_recs(Rec r, bool valid)
{
    const uint32_t d = valid ? r.d : 0u;
    const uint32_t idx = valid ? r.idx : kNoIdx;
    const uint32_t dmax = wave_max_u32(d);
    const uint32_t imin = wave_min_u32((valid && d == dmax) ? idx : kNoIdx);
    const uint64_t who = __builtin_amdgcn_ballot_w64(valid && idx == imin);
    const int src = first_lane(who);
    Rec o;
    o.d = dmax;
    o.idx = imin;
    o.x = rdlane_f(r.x, src);
    o.y = rdlane_f(r.y, src);
    o.z = rdlane_f(r.z, src);
    o.fail = __builtin_amdgcn_ballot_w64(valid && r.fail != 0) != 0 ? 1u : 0u;
    o.pad0 = o.pad1 = 0;
    return o;
}

}  // namespace
}  // namespace fastpoint
#endif
