// Streaming (HBM-bound) kernels: affine quantize / de-quantize (Sec. 2.1 eq. 1-3),
// stand-alone rescale of int32 accumulators, rescaling add (Sec. 3.2.1), weight transpose.
//
// All of them move each byte once.  How fast HBM moves them depends on the order: the kernels walk in tiles
// of 4 x 256 consecutive vectors per workgroup (four independent loads in flight per lane), not with a stride of
// the whole grid between a lane's loads.  Copy of 154 MB each way: 6.0-6.3 TB/s with tiles, 5.2-5.4 with the
// grid-stride order; 4 bytes in, 1 out: 6.7 against 6.3; reading only: 6.9 against 6.1.  Stores are non-temporal
// (quantize of 38.5 M values 35 us, 46 with plain stores); loads are so only for calls whose tensors exceed by far
// what the 256 MB cache could hold for the next pass over them (25 MB copies: 6.0 TB/s with plain loads, 5.5 with
// non-temporal ones; a training step's three passes over 103 MB: 99 us and 106 us).
// Pointers may have any alignment their element type allows (gfx950 loads and stores 16 bytes at any address).
#include <atomic>

#include "qnn_device.h"
#include "tuning.h"

namespace qnn {

constexpr int kThreads = 256, kUnroll = 4, kMaxBlocks = 8192;
constexpr size_t kCacheBytes = (size_t)512 << 20; // inputs and outputs of a call beyond this: non-temporal loads

using f32x4 = float __attribute__((ext_vector_type(4)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using i32x4 = int32_t __attribute__((ext_vector_type(4)));
using u32x2 = uint32_t __attribute__((ext_vector_type(2)));

template <class T, bool NT> __device__ __forceinline__ T load_any(const void *p)
{
    typedef T U __attribute__((aligned(1)));
    const U *q = static_cast<const U *>(p);
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}
template <class T> __device__ __forceinline__ void store_any(void *p, T v)
{
    typedef T U __attribute__((aligned(1)));
    __builtin_nontemporal_store(v, static_cast<U *>(p));
}

// workgroups for `vectors` lane-sized pieces of work
static int grid_for(size_t vectors)
{
    const size_t b = (vectors + kThreads * kUnroll - 1) / (kThreads * kUnroll);
    return (int)(b < 1 ? 1 : (b > (size_t)kMaxBlocks ? (size_t)kMaxBlocks : b));
}

// tiles of kUnroll x kThreads consecutive vectors, every `step`-th from `first` on: item = load(v) for a whole tile, then
// use(v, item)
template <int THREADS = kThreads, class Load, class Use>
__device__ __forceinline__ void for_tiles(size_t nvec, Load load, Use use, uint32_t first, uint32_t step)
{
    constexpr size_t kTile = (size_t)THREADS * kUnroll;
    for (size_t base = (size_t)first * kTile; base < nvec; base += (size_t)step * kTile) {
        const size_t v = base + threadIdx.x;
        if (base + kTile <= nvec) { // uniform
            decltype(load(v)) item[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) item[u] = load(v + u * THREADS);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) use(v + u * THREADS, item[u]);
        } else {
            for (int u = 0; u < kUnroll; ++u)
                if (v + u * THREADS < nvec) use(v + u * THREADS, load(v + u * THREADS));
        }
    }
}
template <int THREADS = kThreads, class Load, class Use> __device__ __forceinline__ void for_tiles(size_t nvec, Load load, Use use)
{
    for_tiles<THREADS>(nvec, load, use, blockIdx.x, gridDim.x);
}

// An element-wise pass: Op::kWidth elements per vector, load / store of a vector, one(i) for the last n % kWidth.
template <class Op, bool NT> __global__ void __launch_bounds__(kThreads) stream_kernel(const Op op_arg, size_t n)
{
    const auto op = op_arg.prepared();
    const size_t nvec = n / Op::kWidth;
    for_tiles(nvec, [&](size_t v) { return op.template load<NT>(v); }, [&](size_t v, auto item) { op.store(v, item); });
    if (blockIdx.x == 0 && threadIdx.x < n - nvec * Op::kWidth) op.one(nvec * Op::kWidth + threadIdx.x);
}

// bytes_per_element: of all inputs and outputs together
template <class Op> static qnn_status launch_stream(const Op &op, size_t n, int bytes_per_element, void *stream)
{
    const dim3 grid((unsigned)grid_for(n / Op::kWidth));
    const hipStream_t s = as_stream(stream);
    if (n * (size_t)bytes_per_element > kCacheBytes) hipLaunchKernelGGL((stream_kernel<Op, true>), grid, dim3(kThreads), 0, s, op, n);
    else hipLaunchKernelGGL((stream_kernel<Op, false>), grid, dim3(kThreads), 0, s, op, n);
    return launch_status(hipGetLastError());
}

// ------------------------------------------------------------------ quantize

__device__ __forceinline__ uint32_t quantize_one(float x, float scale, float lo, float hi, int32_t z)
{
    float t = __fdiv_rn(x, scale);   // one correctly rounded binary32 division
    float r = roundf(t);             // ties away from zero
    r = (t != t) ? 0.0f : r;         // NaN behaves like 0.0
    r = r < lo ? lo : r;
    r = r > hi ? hi : r;
    return (uint32_t)((int32_t)r + z);
}

struct QuantizeOp {
    const float *x;
    uint8_t *q;
    float scale, lo, hi;
    int32_t z;
    static constexpr int kWidth = 4;
    __device__ const QuantizeOp &prepared() const { return *this; }
    template <bool NT> __device__ f32x4 load(size_t v) const { return load_any<f32x4, NT>(x + 4 * v); }
    __device__ void store(size_t v, f32x4 a) const
    {
        store_any<uint32_t>(q + 4 * v, quantize_one(a.x, scale, lo, hi, z) | (quantize_one(a.y, scale, lo, hi, z) << 8) |
                                           (quantize_one(a.z, scale, lo, hi, z) << 16) | (quantize_one(a.w, scale, lo, hi, z) << 24));
    }
    __device__ void one(size_t i) const { q[i] = (uint8_t)quantize_one(x[i], scale, lo, hi, z); }
};

// ------------------------------------------- ranges on the device, dynamic quantization

// Sec. 2.5: activation ranges come from the minimum and maximum of the tensor (their moving average
// across batches during training); Sec. 2.1 turns a range into (scale, zero_point).  Everything stays on
// the device: a reduction with one atomic pair per workgroup on order-preserving integer keys, behind it one
// lane that updates the range and derives the parameters in double precision exactly as
// qnn_choose_qparams does on the host, and a quantize kernel that reads them from memory.
__device__ __forceinline__ uint32_t float_key(float v) // monotonic: a < b  <=>  key(a) < key(b)
{
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// key_min / key_max are all of the state that is work space: scale, zero-point and range are those of the call before until
// the one lane at the end writes them.
__global__ void minmax_init_kernel(qnn_dyn_qparams *st)
{
    st->key_min = 0xffffffffu;
    st->key_max = 0u;
}

// Up to kMinmaxCounted workgroups the last one to arrive finishes the range.  key_min / key_max leave no room to count, so the
// keys and the count are in a slot of the library, claimed on the device for the time of one call; key_min holds its number.
// The host passes the slots round.  A call that finds its own taken (that of 1024 calls ago still runs, or a captured graph
// brings the same number) has none: its workgroup 0 then does it all.
struct RangeSlot {
    uint32_t key_min, key_max, done, busy;
};
constexpr uint32_t kRangeSlots = 1024, kNoSlot = kRangeSlots;
static __device__ RangeSlot g_range_slots[kRangeSlots];

__global__ void minmax_claim_kernel(qnn_dyn_qparams *st, uint32_t number)
{
    RangeSlot &slot = g_range_slots[number < kRangeSlots ? number : 0];
    const bool claimed = number < kRangeSlots && __hip_atomic_exchange(&slot.busy, 1u, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == 0u;
    if (claimed) {
        __hip_atomic_store(&slot.key_min, 0xffffffffu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&slot.key_max, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&slot.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    st->key_min = claimed ? number : kNoSlot;
}

__device__ __forceinline__ double nearest_away_dev(double v) { return v < 0.0 ? -floor(-v + 0.5) : floor(v + 0.5); }

// range update (momentum 0: the batch range; else moving average) and quantizer parameters
__device__ __forceinline__ void finish_range(qnn_dyn_qparams *st, float bmin, float bmax, float momentum, int bits)
{
    if (momentum != 0.0f) { // m * old + (1 - m) * batch, each operation rounded once in double, then to binary32
        const double m = (double)momentum, om = __dsub_rn(1.0, m);
        bmin = (float)__dadd_rn(__dmul_rn(m, (double)st->xmin), __dmul_rn(om, (double)bmin));
        bmax = (float)__dadd_rn(__dmul_rn(m, (double)st->xmax), __dmul_rn(om, (double)bmax));
    }
    st->xmin = bmin, st->xmax = bmax;
    const double lo = fmin((double)bmin, 0.0), hi = fmax((double)bmax, 0.0);
    const double steps = (double)((1 << bits) - 1);
    if (hi - lo == 0.0) {
        st->scale = 1.0f, st->zero_point = 0;
        return;
    }
    const float sc = (float)__ddiv_rn(__dsub_rn(hi, lo), steps);
    double z = nearest_away_dev(__ddiv_rn(-lo, (double)sc));
    z = fmin(fmax(z, 0.0), steps);
    st->scale = sc, st->zero_point = (int32_t)z;
}

__device__ __forceinline__ void finish_keys(qnn_dyn_qparams *st, uint32_t kmin, uint32_t kmax, float momentum, int bits)
{
    const bool any = kmin <= kmax;
    finish_range(st, any ? key_float(kmin) : 0.0f, any ? key_float(kmax) : 0.0f, momentum, bits);
}

__global__ void range_finalize_kernel(qnn_dyn_qparams *st, float momentum, int bits) { finish_keys(st, st->key_min, st->key_max, momentum, bits); }

// Bound by reading x and, behind that, by the atomics: about 10 ns each on one address, and the workgroups end
// together, so that none finds the other's result already there.  One workgroup of 16 waves per CU: 25.7 M values
// in 22 us where 2048 workgroups of 4 waves took 59.  Launches are most of the time of smaller tensors: up to
// kMinmaxAlone values one workgroup does it all, up to kMinmaxCounted workgroups the last one to arrive finishes the range (see
// RangeSlot).  us in a graph / called one by one: one workgroup 65536 values 5.1 / 4.9 (three launches 7.2), 98304 6.3 / 6.2,
// 114688 7.0 / 6.7, 131072 7.6 / 7.4, 163840 8.9 / 8.7; counted 114689 7.2 / 6.8-7.8, 131072 7.0 / 6.9-7.6, 262144 7.5 / 7.0-7.9,
// 524288 7.8 / 7.4-8.2, 1048576 8.7 / 8.4-9.2; three launches 131072 7.4 / 7.5-9.0, 262144 7.5 / 7.5-9.9, 524288 7.8 / 7.6-10.1,
// 1048576 8.5 / 8.3-10.1.  With 256 workgroups the count, one more atomic on one address each, takes 3 us longer than the launch
// it saves.
constexpr int kMinmaxThreads = 1024, kMinmaxBlocks = 256, kMinmaxCounted = 64;
constexpr size_t kMinmaxAlone = (size_t)7 * kMinmaxThreads * kUnroll * 4;
template <bool NT, bool MANY> // MANY: more than kMinmaxCounted workgroups
__global__ void __launch_bounds__(kMinmaxThreads) minmax_kernel(const float *__restrict__ x, size_t n, qnn_dyn_qparams *st, float momentum, int bits)
{
    float lo = INFINITY, hi = -INFINITY; // values that are not finite take no part in the range
    auto take = [&](float v) {
        // one comparison for "finite": the magnitude bits of inf and NaN are the largest
        const bool ok = (__float_as_uint(v) & 0x7fffffffu) < 0x7f800000u;
        lo = fminf(lo, ok ? v : INFINITY), hi = fmaxf(hi, ok ? v : -INFINITY);
    };
    const size_t nvec = n / 4;
    auto load = [&](size_t v) { return load_any<f32x4, NT>(x + 4 * v); };
    auto use = [&](size_t, f32x4 a) { take(a.x), take(a.y), take(a.z), take(a.w); };
    const bool counted = !MANY && gridDim.x > 1;
    const uint32_t number = counted ? st->key_min : 0u; // requested here, used behind the loads
    for_tiles<kMinmaxThreads>(nvec, load, use);
    const bool alone = !MANY && (gridDim.x == 1 || number >= kNoSlot);
    if (alone && gridDim.x > 1) {
        if (blockIdx.x != 0) return;
        for_tiles<kMinmaxThreads>(nvec, load, use, 0, 1);
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nvec * 4) take(x[nvec * 4 + threadIdx.x]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
    }
    __shared__ float s_lo[kMinmaxThreads / 64], s_hi[kMinmaxThreads / 64];
    if ((threadIdx.x & 63) == 0) s_lo[threadIdx.x >> 6] = lo, s_hi[threadIdx.x >> 6] = hi;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < kMinmaxThreads / 64; ++w) lo = fminf(lo, s_lo[w]), hi = fmaxf(hi, s_hi[w]);
    if (alone) {
        finish_range(st, lo <= hi ? lo : 0.0f, lo <= hi ? hi : 0.0f, momentum, bits); // (no finite value at all: 0, 0)
        return;
    }
    RangeSlot *const slot = counted ? &g_range_slots[number] : nullptr;
    uint32_t *const key_min = counted ? &slot->key_min : &st->key_min, *const key_max = counted ? &slot->key_max : &st->key_max;
    if (lo <= hi) { // at least one finite value in this block
        // atomics on one address serialise across the chip: skip them when the value seen so far is
        // already as good (a stale read only costs an atomic that changes nothing)
        const uint32_t klo = float_key(lo), khi = float_key(hi);
        if (klo < __hip_atomic_load(key_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(key_min, klo);
        if (khi > __hip_atomic_load(key_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(key_max, khi);
    }
    if (!counted) return; // range_finalize_kernel comes behind
    // release: this workgroup's keys come before its count; acquire: the last one sees those of all (with a relaxed count, which
    // no rule orders behind the keys, 0.1-0.4 us less)
    if (__hip_atomic_fetch_add(&slot->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1u != gridDim.x) return;
    const uint32_t kmin = __hip_atomic_load(key_min, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t kmax = __hip_atomic_load(key_max, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slot->busy, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    finish_keys(st, kmin, kmax, momentum, bits);
}

// quantize with parameters that live in device memory (8-bit codes)
struct QuantizeWithOp {
    const float *x;
    uint8_t *q;
    const qnn_dyn_qparams *st;
    static constexpr int kWidth = 4;
    __device__ QuantizeOp prepared() const
    {
        const int32_t z = st->zero_point;
        return QuantizeOp{x, q, st->scale, (float)(0 - z), (float)(255 - z), z};
    }
};

// ------------------------------------------------- simulated quantization (training side)

// Sec. 2.4: SimQuant = quantizer followed by de-quantizer (eq. 12-13); in the backward pass the
// quantizer is replaced by a clamp to the representable range, i.e. the incoming gradient passes
// where x_min <= x <= x_max and is zero elsewhere (straight-through estimator, eq. 14-15).
struct SimquantOp {
    const float *x;
    float *y;
    float scale, lo, hi;
    int32_t z;
    static constexpr int kWidth = 4;
    __device__ const SimquantOp &prepared() const { return *this; }
    __device__ float value(float v) const { return __fmul_rn((float)((int32_t)quantize_one(v, scale, lo, hi, z) - z), scale); }
    template <bool NT> __device__ f32x4 load(size_t v) const { return load_any<f32x4, NT>(x + 4 * v); }
    __device__ void store(size_t v, f32x4 a) const { store_any(y + 4 * v, f32x4{value(a.x), value(a.y), value(a.z), value(a.w)}); }
    __device__ void one(size_t i) const { y[i] = value(x[i]); }
};

struct SimquantBackwardOp {
    const float *x, *gy;
    float *gx;
    float xmin, xmax;
    static constexpr int kWidth = 4;
    struct Item {
        f32x4 x, g;
    };
    __device__ const SimquantBackwardOp &prepared() const { return *this; }
    __device__ float value(float v, float g) const { return (v >= xmin && v <= xmax) ? g : 0.0f; } // NaN fails both comparisons: no gradient
    template <bool NT> __device__ Item load(size_t v) const { return {load_any<f32x4, NT>(x + 4 * v), load_any<f32x4, NT>(gy + 4 * v)}; }
    __device__ void store(size_t v, Item t) const
    {
        store_any(gx + 4 * v, f32x4{value(t.x.x, t.g.x), value(t.x.y, t.g.y), value(t.x.z, t.g.z), value(t.x.w, t.g.w)});
    }
    __device__ void one(size_t i) const { gx[i] = value(x[i], gy[i]); }
};

// 16-bit codes (Sec. 3.3 compares activation precisions of 4, 8 and 16 bits): the same arithmetic with
// uint16 storage.
struct QuantizeU16Op {
    const float *x;
    uint16_t *q;
    float scale, lo, hi;
    int32_t z;
    static constexpr int kWidth = 4;
    __device__ const QuantizeU16Op &prepared() const { return *this; }
    template <bool NT> __device__ f32x4 load(size_t v) const { return load_any<f32x4, NT>(x + 4 * v); }
    __device__ void store(size_t v, f32x4 a) const
    {
        store_any(q + 4 * v, u32x2{quantize_one(a.x, scale, lo, hi, z) | (quantize_one(a.y, scale, lo, hi, z) << 16),
                                   quantize_one(a.z, scale, lo, hi, z) | (quantize_one(a.w, scale, lo, hi, z) << 16)});
    }
    __device__ void one(size_t i) const { q[i] = (uint16_t)quantize_one(x[i], scale, lo, hi, z); }
};

// ---------------------------------------------------------------- dequantize

struct DequantizeU16Op {
    const uint16_t *q;
    float *x;
    float scale;
    int32_t z;
    static constexpr int kWidth = 4;
    __device__ const DequantizeU16Op &prepared() const { return *this; }
    __device__ float value(uint32_t c) const { return __fmul_rn((float)((int32_t)c - z), scale); }
    template <bool NT> __device__ u32x2 load(size_t v) const { return load_any<u32x2, NT>(q + 4 * v); }
    __device__ void store(size_t v, u32x2 p) const
    {
        store_any(x + 4 * v, f32x4{value(p.x & 0xffffu), value(p.x >> 16), value(p.y & 0xffffu), value(p.y >> 16)});
    }
    __device__ void one(size_t i) const { x[i] = value(q[i]); }
};

struct DequantizeOp {
    const uint8_t *q;
    float *x;
    float scale;
    int32_t z;
    static constexpr int kWidth = 4;
    __device__ const DequantizeOp &prepared() const { return *this; }
    __device__ float value(uint32_t c) const { return __fmul_rn((float)((int32_t)c - z), scale); }
    template <bool NT> __device__ uint32_t load(size_t v) const { return load_any<uint32_t, NT>(q + 4 * v); }
    __device__ void store(size_t v, uint32_t p) const
    {
        store_any(x + 4 * v, f32x4{value(p & 0xffu), value((p >> 8) & 0xffu), value((p >> 16) & 0xffu), value(p >> 24)});
    }
    __device__ void one(size_t i) const { x[i] = value(q[i]); }
};

// ---------------------------------------------------------------- requantize

// four accumulators of one lane -> four codes.  When every lane of the wave has 1 <= shift <= 20 and
// |acc| < 2^29 the rescale runs in its 7-operation 32-bit form, else in the general 64-bit form.
struct RequantizeArgs {
    const int32_t *acc;
    uint8_t *y;
    const int32_t *mult, *shift;
    size_t total;
    uint32_t channels; // 1: one quantizer for the tensor
    int32_t z_out, act_min, act_max;
};

__device__ __forceinline__ uint32_t requantize_one(const RequantizeArgs &g, int32_t a, int32_t mult, int32_t shift)
{
    // clamp before adding z_out: the rescaled value may sit at the int32 limits
    return (uint32_t)(clamp_i32(g.act_min - g.z_out, g.act_max - g.z_out, rescale_general(a, make_rescale(mult, shift))) + g.z_out);
}

__device__ __forceinline__ uint32_t requantize_four(const RequantizeArgs &g, const i32x4 a, const i32x4 m4, const i32x4 s4,
                                                    const FusedRescale (&f)[4], bool shifts_ok)
{
    bool ok = shifts_ok;
#pragma unroll
    for (int j = 0; j < 4; ++j) ok = ok && a[j] > -(1 << 29) && a[j] < (1 << 29);
    uint32_t packed = 0;
    if (__all(ok)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) packed = shift_into_byte(packed, rescale_fused_w(a[j], f[j]), f[j].n1, j);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) packed |= requantize_one(g, a[j], m4[j], s4[j]) << (8 * j);
    }
    return packed;
}

// FIXED: the tensor has one quantizer, or the channel count divides a row of a tile (4 x 256 elements), so that a
// lane meets the same four channels in all its vectors and holds their parameters; else it looks them up per
// vector (from the cache) and the channel of its first element comes from one multiply-high.
template <bool FIXED, bool NT>
__global__ void __launch_bounds__(kThreads) requantize_kernel(const RequantizeArgs g, uint32_t magic, uint32_t magic_shift)
{
    const size_t nvec = g.total / 4;
    auto params = [&](uint32_t c, i32x4 &m4, i32x4 &s4, FusedRescale (&f)[4]) {
        bool ok = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            m4[j] = g.mult[c], s4[j] = g.shift[c];
            c = c + 1 == g.channels ? 0 : c + 1;
            ok = ok && s4[j] >= 1 && s4[j] <= 20;
            f[j] = make_fused(m4[j], s4[j], 0, g.z_out, g.act_min, g.act_max);
        }
        return ok;
    };
    auto load = [&](size_t v) { return load_any<i32x4, NT>(g.acc + 4 * v); };
    if constexpr (FIXED) {
        i32x4 m4, s4;
        FusedRescale f[4];
        const bool ok = params((threadIdx.x * 4u) % g.channels, m4, s4, f);
        for_tiles(nvec, load, [&](size_t v, i32x4 a) { store_any<uint32_t>(g.y + 4 * v, requantize_four(g, a, m4, s4, f, ok)); });
    } else {
        for_tiles(nvec, load, [&](size_t v, i32x4 a) {
            const size_t i = 4 * v;
            uint32_t c;
            if (g.total < ((size_t)1 << 31)) {
                const uint32_t x = (uint32_t)i;
                c = x - (__umulhi(x, magic) >> magic_shift) * g.channels;
            } else {
                c = (uint32_t)(i % g.channels);
            }
            i32x4 m4, s4;
            FusedRescale f[4];
            const bool ok = params(c, m4, s4, f);
            store_any<uint32_t>(g.y + 4 * v, requantize_four(g, a, m4, s4, f, ok));
        });
    }
    if (blockIdx.x == 0 && threadIdx.x < g.total - nvec * 4) {
        const size_t i = nvec * 4 + threadIdx.x;
        const uint32_t c = (uint32_t)(i % g.channels);
        g.y[i] = (uint8_t)requantize_one(g, g.acc[i], g.mult[c], g.shift[c]);
    }
}

// ---------------------------------------------------------------------- qadd

struct QaddArgs {
    int32_t z_a, mult_a, shift_a, z_b, mult_b, shift_b, left_shift, mult_o, shift_o, z_out, act_min, act_max;
};

// The rescaled value of an input depends only on its 8-bit code, so each block first
// tabulates RESCALE((v - z) * 2^L) for the 256 codes of a and of b in LDS; the streaming
// loop is then two table reads, an add and one rescale per element.
// FUSED: the output rescale may use the 32-bit fused form (1 <= shift_o <= 20 and both tables
// bounded by 2^28, which shift_a, shift_b >= 0 and left_shift <= 20 guarantee).
template <bool FUSED, bool NT>
__global__ void __launch_bounds__(kThreads) qadd_kernel(const uint8_t *__restrict__ a, const uint8_t *__restrict__ b,
                                                        uint8_t *__restrict__ y, size_t n, QaddArgs g)
{
    __shared__ int32_t tab[512];
    const AddParams p = {g.z_a, g.mult_a, g.shift_a, g.z_b, g.mult_b, g.shift_b, g.left_shift, g.mult_o, g.shift_o, g.z_out, g.act_min, g.act_max};
    add_fill_tables(tab, p, threadIdx.x, kThreads);
    __syncthreads();
    const AddOut ao = make_add_out(p);
    struct Item {
        u32x4 a, b;
    };
    const size_t nvec = n / 16;
    for_tiles(nvec, [&](size_t v) { return Item{load_any<u32x4, NT>(a + 16 * v), load_any<u32x4, NT>(b + 16 * v)}; },
              [&](size_t v, Item t) {
                  u32x4 o;
#pragma unroll
                  for (int d = 0; d < 4; ++d) o[d] = add_codes4<FUSED>(t.a[d], t.b[d], tab, ao);
                  store_any(y + 16 * v, o);
              });
    if (blockIdx.x == 0 && threadIdx.x < n - nvec * 16) {
        const size_t i = nvec * 16 + threadIdx.x;
        y[i] = (uint8_t)add_code1<FUSED>(a[i], b[i], tab, ao);
    }
}

// The same with one vector of 4 W codes per lane, requested ahead of the tables.  Small tensors are bound by latencies (a
// lane of the kernel above waits for its tables, then for its codes, and looks up 128 of them one after another, on 16
// workgroups where a layer has 250880), larger ones by how many requests are in flight.  16 codes per lane against the kernel
// above, us: 250880 codes 2.4 and 3.7, 2408448 3.7 and 4.4, 38.5 M 22.7 and 24.1, 51 M 29.5 and 31.7, 77 M 40-44 and 42; then
// the tables of ever more workgroups cost more: 150 M 81 and 77.  8 codes per lane: 250880 2.2, 2408448 3.7, 9.6 M 8.2 (16: 7.3).
// In the general form a workgroup's arithmetic weighs more than its latencies from 12 M codes on: 4.2 M 5.9 and 7.1, 9.6 M 10.6
// and 12.0, 12.6 M 12.2 and 12.2, 25 M 22.7 and 21.5, 50 M 43.3 and 38.8.
constexpr size_t kQaddLanes = (size_t)64 << 20, kQaddLanesGeneral = (size_t)12 << 20;
template <bool FUSED, int W>
__global__ void __launch_bounds__(kThreads) qadd_lane_kernel(const uint8_t *a, const uint8_t *b, uint8_t *y, size_t n, QaddArgs g)
{
    typedef uint32_t Vec __attribute__((ext_vector_type(W)));
    __shared__ int32_t tab[512];
    const AddParams p = {g.z_a, g.mult_a, g.shift_a, g.z_b, g.mult_b, g.shift_b, g.left_shift, g.mult_o, g.shift_o, g.z_out, g.act_min, g.act_max};
    const size_t nvec = n / (4 * W), v = (size_t)blockIdx.x * kThreads + threadIdx.x;
    const size_t at = 4 * W * (v < nvec ? v : nvec - 1); // (the dispatcher guarantees one vector)
    const Vec va = load_any<Vec, false>(a + at), vb = load_any<Vec, false>(b + at);
    asm volatile("" ::: "memory"); // the loads stay here
    add_fill_tables(tab, p, threadIdx.x, kThreads);
    __syncthreads();
    const AddOut ao = make_add_out(p);
    if (v < nvec) {
        Vec o;
#pragma unroll
        for (int d = 0; d < W; ++d) o[d] = add_codes4<FUSED>(va[d], vb[d], tab, ao);
        store_any(y + at, o);
    }
    if (blockIdx.x == 0 && threadIdx.x < n - nvec * (4 * W)) {
        const size_t i = nvec * (4 * W) + threadIdx.x;
        y[i] = (uint8_t)add_code1<FUSED>(a[i], b[i], tab, ao);
    }
}

// ------------------------------------------------------ rescale of uint8 codes (concat)

// Rows of `cols` bytes cut into 16-byte chunks: vector v -> (row, first column).  The last chunk of a row starts at
// cols - 16 (its first `before` bytes are the previous chunk's too), so that rows of any length are whole chunks; rows
// shorter than that are one chunk, byte by byte.
struct RowChunks {
    uint64_t per_row;
    uint32_t magic, magic_shift; // v / per_row for v < 2^31, 2 <= per_row < 2^31; else magic = 0
    int64_t cols;
    bool in_place; // source and destination overlap: every byte is written by the chunk that it belongs to, and once
    __device__ void locate(size_t v, int64_t &row, int64_t &col, int &before) const
    {
        if (per_row == 1) {
            row = (int64_t)v, col = 0;
        } else if (magic && v < ((size_t)1 << 31)) {
            const uint32_t r = __umulhi((uint32_t)v, magic) >> magic_shift;
            row = r, col = (int64_t)((uint32_t)v - r * (uint32_t)per_row) * 16;
        } else {
            row = (int64_t)(v / per_row), col = (int64_t)(v - (size_t)row * per_row) * 16;
        }
        before = 0;
        if (col + 16 > cols && cols >= 16) before = (int)(col - (cols - 16)), col = cols - 16;
    }
};

// Sec. 3.2.1: the inputs of a concatenation carry different quantizers and must be brought to the
// output's before they are laid side by side.  y[m][c] = clamp(z_out + RESCALE(x[m][c] - z_in)) is a
// function of one 8-bit code: a 256-entry byte table per workgroup, one gather per element.  Rows
// have their own pitches, so the destination can be a channel slice of the concatenated tensor.
template <bool NT>
__global__ void __launch_bounds__(kThreads) rescale_u8_kernel(const uint8_t *__restrict__ x, int64_t ldx, uint8_t *__restrict__ y,
                                                              int64_t ldy, size_t chunks, RowChunks rc, int32_t z_in, int32_t mult,
                                                              int32_t shift, int32_t z_out, int32_t act_min, int32_t act_max)
{
    __shared__ uint8_t lut[256];
    {
        const int v = threadIdx.x; // kThreads == 256
        const int32_t r = rescale_general(v - z_in, make_rescale(mult, shift));
        lut[v] = (uint8_t)(clamp_i32(act_min - z_out, act_max - z_out, r) + z_out);
    }
    __syncthreads();
    if (rc.cols < 16) { // uniform
        for (size_t q = (size_t)blockIdx.x * kThreads + threadIdx.x; q < chunks; q += (size_t)gridDim.x * kThreads)
            for (int64_t e = 0; e < rc.cols; ++e) y[(int64_t)q * ldy + e] = lut[x[(int64_t)q * ldx + e]];
        return;
    }
    for_tiles(chunks,
              [&](size_t v) {
                  int64_t m, c;
                  int before;
                  rc.locate(v, m, c, before);
                  return load_any<u32x4, NT>(x + m * ldx + c);
              },
              [&](size_t v, u32x4 a) {
                  int64_t m, c;
                  int before;
                  rc.locate(v, m, c, before);
                  u32x4 o;
#pragma unroll
                  for (int d = 0; d < 4; ++d)
                      o[d] = (uint32_t)lut[a[d] & 0xffu] | ((uint32_t)lut[(a[d] >> 8) & 0xffu] << 8) |
                             ((uint32_t)lut[(a[d] >> 16) & 0xffu] << 16) | ((uint32_t)lut[a[d] >> 24] << 24);
                  uint8_t *const dst = y + m * ldy + c;
                  if (rc.in_place && before > 0) // (the bytes before may have been rescaled already)
                      for (int e = before; e < 16; ++e) dst[e] = (uint8_t)(o[e >> 2] >> (8 * (e & 3)));
                  else store_any(dst, o);
              });
}

// ------------------------------------------------ add behind a product, second-pass form

// y = ADD(y, r) row by row, in place (each 16-byte chunk is read, combined and written by one lane)
template <bool FUSED>
__global__ void __launch_bounds__(kThreads) add_inplace_kernel(uint8_t *y, int64_t ldy, const uint8_t *r, int64_t ldr,
                                                               int64_t M, int64_t N, AddParams p, int vec16)
{
    __shared__ int32_t tab[512];
    add_fill_tables(tab, p, threadIdx.x, kThreads);
    __syncthreads();
    const AddOut ao = make_add_out(p);
    const int64_t chunks_per_row = (N + 15) / 16, total = M * chunks_per_row;
    for (int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x; q < total; q += (int64_t)gridDim.x * kThreads) {
        const int64_t m = q / chunks_per_row;
        const int64_t n = (q - m * chunks_per_row) * 16;
        uint8_t *yp = y + m * ldy + n;
        const uint8_t *rp = r + m * ldr + n;
        if (vec16 && n + 16 <= N) {
            const u32x4 a = *reinterpret_cast<const u32x4 *>(yp), b = *reinterpret_cast<const u32x4 *>(rp);
            u32x4 o;
#pragma unroll
            for (int d = 0; d < 4; ++d) o[d] = add_codes4<FUSED>(a[d], b[d], tab, ao);
            *reinterpret_cast<u32x4 *>(yp) = o;
        } else {
            for (int e = 0; e < 16 && n + e < N; ++e) yp[e] = (uint8_t)add_code1<FUSED>(yp[e], rp[e], tab, ao);
        }
    }
}

// ------------------------------------------------------------------- pack_b

// dst[n][k] = src[k][n], 64x64 byte tiles through LDS so both sides are coalesced
__global__ void __launch_bounds__(kThreads) pack_b_kernel(const int8_t *__restrict__ src, int64_t ld_src, int64_t K,
                                                          int64_t N, int8_t *__restrict__ dst, int64_t ld_dst)
{
    __shared__ int8_t tile[64][65];
    const int64_t k0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int r = ty; r < 64; r += 4) {
        const int64_t k = k0 + r, n = n0 + tx;
        tile[r][tx] = (k < K && n < N) ? src[k * ld_src + n] : (int8_t)0;
    }
    __syncthreads();
    for (int r = ty; r < 64; r += 4) {
        const int64_t n = n0 + r, k = k0 + tx;
        if (n < N && k < K) dst[n * ld_dst + k] = tile[tx][r];
    }
}

static bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

qnn_status launch_add_inplace(uint8_t *y, int64_t ldy, const uint8_t *r, int64_t ldr, int64_t M, int32_t N,
                              const AddParams &p, hipStream_t s)
{
    int64_t rows = M, cols = N;
    if (ldy == N && ldr == N) rows = 1, cols = M * (int64_t)N, ldy = ldr = cols; // dense: one long row, whole chunks throughout
    const int vec16 = aligned(y, 16) && aligned(r, 16) && (rows == 1 || ((ldy % 16) == 0 && (ldr % 16) == 0));
    const size_t chunks = (size_t)rows * (size_t)((cols + 15) / 16);
    size_t blocks = (chunks + kThreads * 2 - 1) / (kThreads * 2);
    const int grid = (int)(blocks > 256 * 16 ? 256 * 16 : blocks);
    const bool fused = p.shift_o >= 1 && p.shift_o <= 20 && p.shift_m >= 0 && p.shift_r >= 0 && p.left_shift <= 20;
    if (fused) hipLaunchKernelGGL((add_inplace_kernel<true>), dim3(grid), dim3(kThreads), 0, s, y, ldy, r, ldr, rows, cols, p, vec16);
    else hipLaunchKernelGGL((add_inplace_kernel<false>), dim3(grid), dim3(kThreads), 0, s, y, ldy, r, ldr, rows, cols, p, vec16);
    return launch_status(hipGetLastError());
}

} // namespace qnn

using namespace qnn;

extern "C" {

qnn_status qnn_quantize(const float *x, uint8_t *q, size_t n, float scale, int32_t zero_point, int32_t qmin,
                        int32_t qmax, void *stream)
{
    if (!(scale > 0.0f) || __builtin_isinf(scale)) return QNN_EINVAL;
    if (qmin < 0 || qmax > 255 || qmin > qmax || zero_point < qmin || zero_point > qmax) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !q) return QNN_EINVAL;
    return launch_stream(QuantizeOp{x, q, scale, (float)(qmin - zero_point), (float)(qmax - zero_point), zero_point}, n, 5, stream);
}

qnn_status qnn_dequantize(const uint8_t *q, float *x, size_t n, float scale, int32_t zero_point, void *stream)
{
    if (!(scale > 0.0f) || __builtin_isinf(scale) || zero_point < 0 || zero_point > 255) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !q) return QNN_EINVAL;
    return launch_stream(DequantizeOp{q, x, scale, zero_point}, n, 5, stream);
}

qnn_status qnn_quantize_u16(const float *x, uint16_t *q, size_t n, float scale, int32_t zero_point, int32_t qmin,
                            int32_t qmax, void *stream)
{
    if (!(scale > 0.0f) || __builtin_isinf(scale)) return QNN_EINVAL;
    if (qmin < 0 || qmax > 65535 || qmin > qmax || zero_point < qmin || zero_point > qmax) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !q) return QNN_EINVAL;
    return launch_stream(QuantizeU16Op{x, q, scale, (float)(qmin - zero_point), (float)(qmax - zero_point), zero_point}, n, 6, stream);
}

qnn_status qnn_dequantize_u16(const uint16_t *q, float *x, size_t n, float scale, int32_t zero_point, void *stream)
{
    if (!(scale > 0.0f) || __builtin_isinf(scale) || zero_point < 0 || zero_point > 65535) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !q) return QNN_EINVAL;
    return launch_stream(DequantizeU16Op{q, x, scale, zero_point}, n, 6, stream);
}

qnn_status qnn_requantize(const int32_t *acc, uint8_t *y, size_t rows, size_t channels, const int32_t *mult,
                          const int32_t *shift, int per_channel, int32_t z_out, int32_t act_min, int32_t act_max,
                          void *stream)
{
    if (!acc || !y || !mult || !shift || rows == 0 || channels == 0 || channels > 0x7fffffffu) return QNN_EINVAL;
    if (bad_out_range(z_out, act_min, act_max)) return QNN_EINVAL;
    const size_t total = rows * channels;
    const RequantizeArgs g = {acc, y, mult, shift, total, per_channel ? (uint32_t)channels : 1u, z_out, act_min, act_max};
    uint32_t magic, magic_shift;
    fast_division(g.channels, magic, magic_shift);
    const bool fixed = (4 * kThreads) % g.channels == 0, nt = total * 5 > kCacheBytes;
    const dim3 grid((unsigned)grid_for(total / 4));
    const hipStream_t s = as_stream(stream);
    if (fixed && nt) hipLaunchKernelGGL((requantize_kernel<true, true>), grid, dim3(kThreads), 0, s, g, magic, magic_shift);
    else if (fixed) hipLaunchKernelGGL((requantize_kernel<true, false>), grid, dim3(kThreads), 0, s, g, magic, magic_shift);
    else if (nt) hipLaunchKernelGGL((requantize_kernel<false, true>), grid, dim3(kThreads), 0, s, g, magic, magic_shift);
    else hipLaunchKernelGGL((requantize_kernel<false, false>), grid, dim3(kThreads), 0, s, g, magic, magic_shift);
    return launch_status(hipGetLastError());
}

qnn_status qnn_minmax(const float *x, size_t n, float momentum, int bits, qnn_dyn_qparams *state, void *stream)
{
    if (!state || (n && !x) || bits < 2 || bits > 16 || !(momentum >= 0.0f) || !(momentum < 1.0f)) return QNN_EINVAL;
    const hipStream_t s = as_stream(stream);
    const size_t tiles = (n / 4 + kMinmaxThreads * kUnroll - 1) / (kMinmaxThreads * kUnroll);
    const dim3 grid((unsigned)(n <= kMinmaxAlone ? 1 : (tiles < kMinmaxBlocks ? tiles : kMinmaxBlocks)));
    const bool counted = grid.x > 1 && grid.x <= kMinmaxCounted;
    if (counted) {
        static std::atomic<uint32_t> calls{0};
        const uint32_t number = tuning().range_slot >= 0 ? (uint32_t)tuning().range_slot : calls.fetch_add(1, std::memory_order_relaxed) % kRangeSlots;
        hipLaunchKernelGGL(minmax_claim_kernel, dim3(1), dim3(1), 0, s, state, number);
        // without it the reduction would take whatever the state holds for its slot
        if (const qnn_status st = launch_status(hipGetLastError()); st != QNN_OK) return st;
    } else if (grid.x > 1) hipLaunchKernelGGL(minmax_init_kernel, dim3(1), dim3(1), 0, s, state);
    static_assert((kMinmaxBlocks + 1) * (size_t)kMinmaxThreads * kUnroll * 16 < kCacheBytes, "only launches of many workgroups exceed the cache");
    if (n * 4 > kCacheBytes) hipLaunchKernelGGL((minmax_kernel<true, true>), grid, dim3(kMinmaxThreads), 0, s, x, n, state, momentum, bits);
    else if (grid.x > kMinmaxCounted) hipLaunchKernelGGL((minmax_kernel<false, true>), grid, dim3(kMinmaxThreads), 0, s, x, n, state, momentum, bits);
    else hipLaunchKernelGGL((minmax_kernel<false, false>), grid, dim3(kMinmaxThreads), 0, s, x, n, state, momentum, bits);
    if (grid.x > kMinmaxCounted) hipLaunchKernelGGL(range_finalize_kernel, dim3(1), dim3(1), 0, s, state, momentum, bits);
    return launch_status(hipGetLastError());
}

qnn_status qnn_quantize_with(const float *x, uint8_t *q, size_t n, const qnn_dyn_qparams *state, void *stream)
{
    if (!state) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !q) return QNN_EINVAL;
    return launch_stream(QuantizeWithOp{x, q, state}, n, 5, stream);
}

qnn_status qnn_quantize_dynamic(const float *x, uint8_t *q, size_t n, qnn_dyn_qparams *state, void *stream)
{
    if (n && (!x || !q)) return QNN_EINVAL;
    const qnn_status st = qnn_minmax(x, n, 0.0f, 8, state, stream);
    return st != QNN_OK ? st : qnn_quantize_with(x, q, n, state, stream);
}

qnn_status qnn_simquant(const float *x, float *y, size_t n, float scale, int32_t zero_point, int32_t qmin, int32_t qmax,
                        void *stream)
{
    if (!(scale > 0.0f) || __builtin_isinf(scale) || qmin < 0 || qmax > 65535 || qmin > qmax) return QNN_EINVAL;
    if (zero_point < qmin || zero_point > qmax) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !y) return QNN_EINVAL;
    return launch_stream(SimquantOp{x, y, scale, (float)(qmin - zero_point), (float)(qmax - zero_point), zero_point}, n, 8, stream);
}

qnn_status qnn_simquant_backward(const float *x, const float *grad_y, float *grad_x, size_t n, float scale,
                                 int32_t zero_point, int32_t qmin, int32_t qmax, void *stream)
{
    if (!(scale > 0.0f) || __builtin_isinf(scale) || qmin < 0 || qmax > 65535 || qmin > qmax) return QNN_EINVAL;
    if (zero_point < qmin || zero_point > qmax) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!x || !grad_y || !grad_x) return QNN_EINVAL;
    // the ends of the representable range are the de-quantized extreme codes (one binary32 product each)
    const float xmin = (float)(qmin - zero_point) * scale, xmax = (float)(qmax - zero_point) * scale;
    return launch_stream(SimquantBackwardOp{x, grad_y, grad_x, xmin, xmax}, n, 12, stream);
}

qnn_status qnn_rescale_u8(const uint8_t *x, int64_t ldx, int32_t z_in, int32_t mult, int32_t shift, int32_t z_out,
                          int32_t act_min, int32_t act_max, uint8_t *y, int64_t ldy, int64_t rows, int64_t cols, void *stream)
{
    if (rows < 0 || cols < 0 || z_in < 0 || z_in > 255 || shift < -31 || shift > 31) return QNN_EINVAL;
    if (bad_out_range(z_out, act_min, act_max)) return QNN_EINVAL;
    if (rows == 0 || cols == 0) return QNN_OK;
    if (!x || !y || ldx < cols || ldy < cols) return QNN_EINVAL;
    int64_t r = rows, c = cols;
    if (ldx == cols && ldy == cols) r = 1, c = rows * cols, ldx = ldy = c; // dense: one long row, whole chunks throughout
    RowChunks rc = {};
    rc.per_row = (uint64_t)(c + 15) / 16, rc.cols = c;
    if (rc.per_row <= 0x7fffffff) fast_division((uint32_t)rc.per_row, rc.magic, rc.magic_shift);
    rc.in_place = x < y + (r - 1) * ldy + c && y < x + (r - 1) * ldx + c;
    const size_t chunks = (size_t)r * rc.per_row;
    const dim3 grid((unsigned)grid_for(chunks));
    const hipStream_t s = as_stream(stream);
    if ((size_t)rows * (size_t)cols * 2 > kCacheBytes)
        hipLaunchKernelGGL(rescale_u8_kernel<true>, grid, dim3(kThreads), 0, s, x, ldx, y, ldy, chunks, rc, z_in, mult, shift, z_out, act_min, act_max);
    else
        hipLaunchKernelGGL(rescale_u8_kernel<false>, grid, dim3(kThreads), 0, s, x, ldx, y, ldy, chunks, rc, z_in, mult, shift, z_out, act_min, act_max);
    return launch_status(hipGetLastError());
}

qnn_status qnn_qadd(const uint8_t *a, int32_t z_a, int32_t mult_a, int32_t shift_a, const uint8_t *b, int32_t z_b,
                    int32_t mult_b, int32_t shift_b, int32_t left_shift, int32_t mult_o, int32_t shift_o,
                    int32_t z_out, int32_t act_min, int32_t act_max, uint8_t *y, size_t n, void *stream)
{
    if (left_shift < 0 || left_shift > 22 || z_a < 0 || z_a > 255 || z_b < 0 || z_b > 255) return QNN_EINVAL;
    if (bad_out_range(z_out, act_min, act_max)) return QNN_EINVAL;
    auto bad_shift = [](int32_t s) { return s < -31 || s > 31; };
    if (bad_shift(shift_a) || bad_shift(shift_b) || bad_shift(shift_o)) return QNN_EINVAL;
    if (n == 0) return QNN_OK;
    if (!a || !b || !y) return QNN_EINVAL;
    QaddArgs g = {z_a, mult_a, shift_a, z_b, mult_b, shift_b, left_shift, mult_o, shift_o, z_out, act_min, act_max};
    const bool fused = shift_o >= 1 && shift_o <= 20 && shift_a >= 0 && shift_b >= 0 && left_shift <= 20;
    const hipStream_t s = as_stream(stream);
    if (n >= 8 && n <= (fused ? kQaddLanes : kQaddLanesGeneral)) { // see kQaddLanes; 8 codes per lane while that is no more than a workgroup per CU
        const bool narrow = n <= (size_t)256 * kThreads * 8;
        const dim3 grid((unsigned)((n / (narrow ? 8 : 16) + kThreads - 1) / kThreads));
        if (fused && narrow) hipLaunchKernelGGL((qadd_lane_kernel<true, 2>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
        else if (fused) hipLaunchKernelGGL((qadd_lane_kernel<true, 4>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
        else if (narrow) hipLaunchKernelGGL((qadd_lane_kernel<false, 2>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
        else hipLaunchKernelGGL((qadd_lane_kernel<false, 4>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
        return launch_status(hipGetLastError());
    }
    const dim3 grid((unsigned)grid_for(n / 16));
    const bool nt = n * 3 > kCacheBytes;
    if (fused && nt) hipLaunchKernelGGL((qadd_kernel<true, true>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
    else if (fused) hipLaunchKernelGGL((qadd_kernel<true, false>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
    else if (nt) hipLaunchKernelGGL((qadd_kernel<false, true>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
    else hipLaunchKernelGGL((qadd_kernel<false, false>), grid, dim3(kThreads), 0, s, a, b, y, n, g);
    return launch_status(hipGetLastError());
}

qnn_status qnn_pack_b(const int8_t *src, int64_t ld_src, int64_t K, int64_t N, int8_t *dst, int64_t ld_dst,
                      void *stream)
{
    if (!src || !dst || K <= 0 || N <= 0 || ld_src < N || ld_dst < K) return QNN_EINVAL;
    if ((N + 63) / 64 > 0x7fffffff || (K + 63) / 64 > 65535) return QNN_EINVAL;
    dim3 grid((unsigned)((N + 63) / 64), (unsigned)((K + 63) / 64));
    hipLaunchKernelGGL(pack_b_kernel, grid, dim3(kThreads), 0, as_stream(stream), src, ld_src, K, N, dst, ld_dst);
    return launch_status(hipGetLastError());
}

} // extern "C"
