// Host-only build of libkvp's state machine: the kernel launchers are replaced by stubs, everything else --
// validation, layout, the per-layer state machine, the launch planning of plan.cpp -- is the real code, compiled
// with -fsanitize=address,undefined.  A dry-run cache never calls a launcher.  While the driver records, the launchers
// note what they would launch, for how many layers, and check the divisions by multiplication that their kernels
// would make; otherwise they refuse.
#include <cstdio>
#include <cstdlib>

#include "kvp_internal.h"
#include "stubs.h"

std::vector<Launch>* recorded = nullptr;

namespace {
hipError_t note(const char* kernel, int layers) {
  if (!recorded) return hipErrorNotSupported;
  recorded->push_back(Launch{kernel, layers});
  return hipSuccess;
}
// a division by multiplication, for every dividend below `end`, as the kernel makes it
template <class Magic>
void check_quotients(const char* kernel, int end, int d, Magic magic) {
  if (!recorded) return;
  for (int w = 0; w < end; ++w)
    if (kvp::quotient((unsigned)w, magic) != (unsigned)(w / d)) {
      std::fprintf(stderr, "%s: %d / %d is not %u\n", kernel, w, d, kvp::quotient((unsigned)w, magic));
      std::exit(1);
    }
}
hipError_t note_nothing() { return recorded ? hipSuccess : hipErrorNotSupported; }
}  // namespace

namespace kvp {

hipError_t launch_attention(const AttnArgs& a, int, hipStream_t) {
  if (a.variant == kAttnSplit32 || a.variant == kAttnSplit64) {
    check_quotients("attention_split, row tiles", a.total_work, a.n_row_tiles, a.tiles_magic);
    check_quotients("attention_split, group", a.n_q_heads, a.group, a.group_magic);
  } else {
    check_quotients("attention, row tiles", a.total_work, a.n_row_tiles, Divisor{a.tiles_magic, a.tiles_shift});
    check_quotients("attention, group", a.n_q_heads, a.group, Divisor{a.group_magic, a.group_shift});
  }
  return note(a.key_score_wgs > 0 ? "attention+keys" : "attention", a.g.n_layers);
}
hipError_t launch_colsum(const ColsumArgs& a, int, hipStream_t) {
  check_quotients("colsum, workgroups of a head", a.total_work, a.wgs_per_head, a.wgs_magic);
  return note("colsum", a.g.n_layers);
}
hipError_t launch_select(const SelectArgs& a, int, hipStream_t) {
  // the kernels that select.hip is built for
  if (a.threads != 1024 && (a.threads != 512 || a.items > (a.head_dim == 64 ? 4 : 2))) {
    std::fprintf(stderr, "select: %d threads, %d candidates each at d %d\n", a.threads, a.items, a.head_dim);
    std::exit(1);
  }
  check_quotients("select, groups", a.n_partials + a.groups, a.groups, a.groups_magic);
  return note(a.keydiff ? "keys+select" : "select", a.g.n_layers);
}
hipError_t launch_move(const CompactArgs& a, hipStream_t) { return note("move", a.g.n_layers); }
hipError_t launch_init(int32_t*, float*, size_t, const Seg*, int, Seg*, unsigned long long*, hipStream_t) { return note_nothing(); }
hipError_t launch_rowstat(RowstatArgs a, int, hipStream_t) { return note("rowstat", a.g.n_layers); }
hipError_t launch_keydiff(KeydiffArgs a, int, hipStream_t) { return note("keydiff", a.g.n_layers); }
hipError_t launch_decode(const DecodeArgs&, int, hipStream_t) { return note("decode", 1); }
hipError_t decode_static_scratch(float** ptr, size_t* n_floats) {
  *ptr = nullptr;
  *n_floats = 0;
  return note_nothing();
}
hipError_t prepare_attention() { return note_nothing(); }
hipError_t prepare_select() { return note_nothing(); }

}  // namespace kvp

// the HIP runtime calls kvp.cpp makes (events, stream waits): never reached, neither by a dry-run cache nor on one stream
extern "C" {
hipError_t hipEventCreate(hipEvent_t*) { return hipErrorNotSupported; }
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipErrorNotSupported; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipErrorNotSupported; }
}
