// Constants and device helpers shared by the kernel files (internal).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace pc {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#define PC_NEG_INF (-__builtin_inff())
#define PC_LOG2E 1.4426950408889634f
// Sum-layer terms are theta * exp(value - running maximum + PC_UP).  The maximum is taken over the values alone (as in
// Alg. 1 / Alg. 4), so without the upward shift a term with a large weight whose value lies 87 nats below that of a
// child with a weight near FLT_MIN would be flushed to zero although it dominates the sum.  With it every term or
// factor that underflows is at least e^-20 smaller than the largest term kept, and nothing can overflow.  The shift
// is kept small because the result is  maximum - PC_UP + log(sum): the larger the two cancelling parts, the larger
// the absolute rounding error of a log-probability near zero.
#define PC_UP 20.0f
// Rescaling an accumulator when the running maximum grows by -delta: the factor exp(delta) itself may leave the
// fp32 range where accumulator * factor does not (the accumulator can be as large as e^28 times the term count),
// so the factor is applied as two multiplications by exp(delta / 2); below delta = -174 the result is nil anyway.
__device__ inline float pc_half_scale(float delta) { return __expf(0.5f * fmaxf(delta, -174.0f)); }

// buffer descriptors: raw (stride 0), 2 GiB window from the base, 32-bit data format
#define PC_BUF_RANGE 0x7fffffff
#define PC_BUF_FLAGS 0x00020000

}  // namespace pc
