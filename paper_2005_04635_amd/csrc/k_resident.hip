// On-chip iteration for small states (n <= 14): one workgroup loads the whole state into registers once, runs all k
// iterations of Algorithm 5's loop body there (oracle sign, sum, update), and writes it back once.  The only
// synchronisation per iteration is the one workgroup barrier of the sum, so small searches (e.g. n = 10, 25
// iterations) cost one launch instead of 2k passes over memory.
//
// What bounds an iteration is the workgroup's sum (0.23 us with 256 threads, 0.30 with 512, two waves per SIMD) and
// the update's instructions.  So the workgroup is as small as its registers allow without making the update the
// larger part: one wave up to 256 vectors, whose sum needs no barrier at all, 256 threads up to 1024, then 512 with
// up to 32 vectors per thread.  On MI355X, whole searches with reset, against 1024 threads for every size with a sign
// factor on every amplitude: n = 10 binary64, 25 iterations and 10^4 shots 35 -> 15 us; n = 13 complex64, 41 iterations
// 82 -> 37 us.
#include "held.h"

namespace grover {
namespace {

struct ResidentArgs {
    void *state;
    uint64_t nvec;
    double scale;  // 2 / N, a power of two: S * scale rounds as 2S / N
    const uint64_t *marks;
    uint64_t m;
    uint64_t iters;
};

// NE vectors per thread of a B-thread workgroup; U32: the update in binary32 from 2S/N rounded to binary32
// (complex64 only), otherwise binary64.
template <class T, bool U32, int B, int NE>
__global__ __launch_bounds__(B) void resident_iterate_kernel(ResidentArgs a)
{
    using V = typename T::vec;
    constexpr bool kWide = std::is_same<T, C64>::value && !U32 && NE <= 16;
    __shared__ TeamShared<B> sh;
    __shared__ uint32_t words[WaveMarks<NE, B, T::EPV>::kWords];
    unsigned parity = 0;
    (void)held_run<T, U32, kWide, NE, NE, B, true>(
        static_cast<V *>(a.state), 0, a.nvec, a.marks, a.m, a.iters, a.scale, V{}, words,
        static_cast<V *>(nullptr),
        []() { return true; },
        [&](double &r, double &i) {
            block_allsum<B>(r, i, parity++, sh);
            return true;
        });
}

template <class T, bool U32, int B, int NE>
const void *kernel()
{
    return reinterpret_cast<const void *>(&resident_iterate_kernel<T, U32, B, NE>);
}

// The kernel for a state of nvec vectors (a power of two, at most 2^14 / EPV) and its workgroup size.
template <class T, bool U32 = false>
const void *pick(uint64_t nvec, unsigned &block)
{
    block = nvec <= 256 ? 64 : nvec <= 1024 ? 256 : 512;
    switch (nvec) {
    case 128: return kernel<T, U32, 64, 2>();
    case 256: return kernel<T, U32, 64, 4>();
    case 512: return kernel<T, U32, 256, 2>();
    case 1024: return kernel<T, U32, 256, 4>();
    case 2048: return kernel<T, U32, 512, 4>();
    case 4096: return kernel<T, U32, 512, 8>();
    case 8192: return kernel<T, U32, 512, 16>();
    case 16384:
        if constexpr (T::EPV == 1)
            return kernel<T, U32, 512, 32>();
        return nullptr;
    default: return nvec <= 64 ? kernel<T, U32, 64, 1>() : nullptr;
    }
}

}  // namespace

unsigned resident_block(const grover_ctx *c)
{
    unsigned block = 0;
    (void)pick<C64>(c->N / elems_per_vec(c->dtype), block);
    return block;
}

hipError_t launch_resident_iterate(grover_ctx *c, uint64_t k)
{
    ResidentArgs a;
    a.state = c->state;
    a.nvec = c->N / elems_per_vec(c->dtype);
    a.scale = 2.0 / double(c->N);
    a.marks = c->marks_dev;
    a.m = c->marks.size();
    a.iters = k;
    const void *fn = nullptr;
    unsigned block = 0;
    switch (c->dtype) {
    case GROVER_F64_REAL: fn = pick<F64Real>(a.nvec, block); break;
    case GROVER_C64: fn = c->update == GROVER_UPDATE_F32 ? pick<C64, true>(a.nvec, block) : pick<C64>(a.nvec, block); break;
    case GROVER_C128: fn = pick<C128>(a.nvec, block); break;
    }
    if (!fn)
        return hipErrorInvalidValue;
    void *args[] = {&a};
    return hipLaunchKernel(fn, dim3(1), dim3(block), args, 0, c->stream);
}

}  // namespace grover
