// ddamg_apply_D_noalloc: the canonical-layout Wilson-clover apply in FP64 and
// FP32 for callers that cannot allocate device memory (code under HIP graph
// capture, tight serving loops, harnesses that forbid hipMalloc).  It is the
// kernel of ddamg_apply_D, which reads and writes canonical fields directly, so
// there is no staging memory and calls on several streams or threads do not
// meet.  The batch size it accepts is still the one that two native fields per
// right-hand side in DDAMG_NOALLOC_SCRATCH_BYTES allow: callers have it as an
// EINVAL.
#include "handles.h"

using namespace ddamg;

extern "C" int ddamg_apply_D_noalloc(ddamg_ctx ctx, const void* in, void* out, int nrhs, int prec,
                                     void* stream) {
  return guarded([&] {
    DD_REQUIRE(ctx && ctx->c, "null context");
    DD_REQUIRE(in && out && in != out, "in/out must be distinct device pointers");
    DD_REQUIRE(nrhs >= 1, "nrhs must be >= 1");
    DD_REQUIRE(prec == DDAMG_F64 || prec == DDAMG_F32, "prec must be DDAMG_F64 or DDAMG_F32");
    const Context& c = *ctx->c;
    const size_t need = 2 * (size_t)nrhs * c.g.V * 12 * (prec == DDAMG_F64 ? sizeof(double2) : sizeof(float2));
    DD_REQUIRE(need <= (size_t)DDAMG_NOALLOC_SCRATCH_BYTES,
               "ddamg_apply_D_noalloc: " + std::to_string(nrhs) + " field(s) of " + std::to_string(c.g.V) +
                   " sites count as " + std::to_string(need) + " bytes of staging, more than the " +
                   std::to_string((size_t)DDAMG_NOALLOC_SCRATCH_BYTES) + " accepted");
    const double2* i = static_cast<const double2*>(in);
    double2* o = static_cast<double2*>(out);
    const hipStream_t s = as_stream(stream);
    if (prec == DDAMG_F64) dslash_canonical<double>(c.g, c.view<double>(), i, o, s, nrhs);
    else dslash_canonical<float>(c.g, c.view<float>(), i, o, s, nrhs);
  });
}
