// The launch decisions of the library's host code as plain C functions, for the
// tests of those decisions.  Host code only: no HIP call is made and no pointer of
// a task is followed.
#include "../../paper_2007_01277_amd/csrc/hf_runtime.hpp"

static hf::DevTask prepared(const hf_task* t, bool own) {
  hf::DevTask d;
  if (hf::prepare(t, nullptr, own, &d) != HF_OK) std::abort();
  return d;
}

extern "C" {

// Workgroups of `block` lanes by default for a task that has `waves` wavefronts of
// each, where `resident` of them fit the chip's `num_cus` compute units.  own: its
// scratch is the library's.
uint32_t plan_wgs(const hf_task* t, int own, int waves, int block, int resident, int num_cus) {
  const hf::DevTask d = prepared(t, own != 0);
  return hf::default_wgs(t, d, waves, block, resident, num_cus);
}

// Workgroups that find work.
int64_t plan_useful(const hf_task* t, int waves) {
  const hf::DevTask d = prepared(t, true);
  return hf::useful_wgs(t, d, waves);
}

// Bytes of a task's scratch in the library's own memory, and of an arena slot
// allocated for `bytes`.
int64_t plan_own_scratch(const hf_task* t) { return (int64_t)hf::own_scratch_bytes(t); }
int64_t plan_slot(int64_t bytes) { return (int64_t)hf::slot_bytes((size_t)bytes); }

// Path of an upsample: 2 rows, 1 places, 0 pointwise.
int plan_upsample_path(const hf_task* t) {
  const hf::DevTask d = prepared(t, true);
  return d.up.row2 ? 2 : d.up.places ? 1 : 0;
}

}  // extern "C"
