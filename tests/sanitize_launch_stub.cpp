// Launchers for host-only builds of the C entry points (tests/test_sanitizers.py,
// tests/test_dispatch.py): they launch nothing, count their calls and report a
// launch error, so an argument the checks wrongly accept shows up as
// ATTN_ELAUNCH and as a nonzero count, and they keep the kernel form that the
// last call asked for.
#include <stddef.h>
#include <stdint.h>

#include "attn_params.h"

static int g_launches = 0;
static int g_layout = -1, g_unit = -1, g_k_lds = -1, g_parts = -1;

namespace h15 {

int launch_fwd(const Params& p, int, int, int, int, void*, bool) { return g_layout = p.layout, ++g_launches, 1; }
int launch_probe_fill(float*, float*, uint32_t*, size_t, void*) { return ++g_launches, 1; }
int launch_decode(const DecParams& p, int, int, int, int, void*, bool) {
  g_unit = p.unit, g_k_lds = p.k_lds, g_parts = p.nsplit;
  return ++g_launches, 1;
}
// the built-in decode workspace: the library's stated size, no address
size_t scratch_capacity() { return (size_t)16 << 20; }
int scratch_address(void*, void**) { return ++g_launches, 1; }

}  // namespace h15

extern "C" int h15_stub_launches(void) { return g_launches; }
// of the last forward call: its layout; of the last decode call: keys of a
// wave and round, whether K goes through LDS, number of parts
extern "C" int h15_stub_layout(void) { return g_layout; }
extern "C" int h15_stub_unit(void) { return g_unit; }
extern "C" int h15_stub_k_lds(void) { return g_k_lds; }
extern "C" int h15_stub_parts(void) { return g_parts; }
