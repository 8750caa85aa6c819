// host_containers.cpp -- host side of the container calls: capacity,
// reserve, resize, push_back, rebind, element writes and removal by
// overwriting with the last particle.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <map>
#include <string>
#include <tuple>
#include <vector>

#include "host_internal.h"

using namespace soax;
using namespace soax::host;

// ----------------------------------------------------------- containers

namespace {

// Move an owned set into buffers for `cap` particles, keeping its n
// particles in both copies.  Synchronises `s` before freeing the old buffers.
soax_status grow(soax_set* set, int64_t cap, hipStream_t s) {
  void* nsoa_block = nullptr;
  void* naos = nullptr;
  std::vector<void*> nsoa;
  soax_status st = alloc_owned(set->L, cap, &nsoa_block, nsoa, &naos);
  if (st) return st;
  hipError_t e = hipSuccess;
  if (set->n > 0) {
    for (const Field& f : set->L.f)
      for (int c = 0; c < f.dim && e == hipSuccess; ++c) {
        const int a = f.first_array + c;
        e = launch_copy16(nsoa[a], set->soa[a], set->n * f.es, s);
      }
    if (e == hipSuccess) e = launch_copy16(naos, set->aos, set->n * set->L.stride, s);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    (void)hipFree(nsoa_block);
    (void)hipFree(naos);
    return hip_fail(e, "copy into the grown buffers");
  }
  (void)hipFree(set->owned_soa);
  (void)hipFree(set->owned_aos);
  set->owned_soa = nsoa_block;
  set->owned_aos = naos;
  set->soa = nsoa;
  set->aos = static_cast<char*>(naos);
  set->cap = cap;
  set->aosoa = nullptr;  // the AoSoA table names the old SoA arrays
  ++set->generation;
  return finish_set(set);  // the stream is idle: the new table can be uploaded
}

// Room for `need` particles: bound sets must already have it; owned sets
// grow to max(need, 2 * capacity), at most 2^31-1.
soax_status ensure_capacity(soax_set* set, int64_t need, hipStream_t s) {
  if (need <= set->cap) return SOAX_OK;
  if (!set->owns)
    return fail(SOAX_E_STATE, "a bound set holds at most %lld particles (asked for %lld)",
                static_cast<long long>(set->cap), static_cast<long long>(need));
  return grow(set, std::max(need, std::min(2 * set->cap, kMaxParticles)), s);
}

// New size (host state only: the kernels take n as an argument).
soax_status set_size(soax_set* set, int64_t n) {
  set->n = n;
  set->xpose_host.n = n;
  ++set->generation;
  return SOAX_OK;
}

// Width in bytes of the moves of one AoS record: the widest of 16, 8, 4
// that divides the stride and the buffer's alignment.
int record_word(const soax_set* set) {
  const uintptr_t a = reinterpret_cast<uintptr_t>(set->aos);
  for (int w : {16, 8, 4})
    if (set->L.stride % w == 0 && a % w == 0) return w;
  return 1;
}

struct DevBuf {  // stream-ordered scratch, released on the same stream
  void* p = nullptr;
  hipStream_t s = nullptr;
  hipError_t alloc(size_t bytes, hipStream_t st) {
    s = st;
    return bytes ? hipMallocAsync(&p, bytes, st) : hipSuccess;
  }
  ~DevBuf() {
    if (p) (void)hipFreeAsync(p, s);
  }
};

}  // namespace

extern "C" {

soax_status soax_capacity(const soax_set* set, int64_t* n, int64_t* capacity) {
  if (!set) return fail(SOAX_E_ARG, "set is NULL");
  if (n) *n = set->n;
  if (capacity) *capacity = set->cap;
  return SOAX_OK;
}

soax_status soax_reserve(soax_set* set, int64_t capacity, void* stream) {
  if (!set) return fail(SOAX_E_ARG, "set is NULL");
  soax_status st;
  if ((st = check_n(set->L, capacity))) return st;
  if (capacity <= set->cap) return SOAX_OK;
  const hipStream_t s = as_stream(stream);
  if (!set->owns)
    return fail(SOAX_E_STATE, "a bound set holds at most %lld particles",
                static_cast<long long>(set->cap));
  return grow(set, capacity, s);
}

soax_status soax_resize(soax_set* set, int64_t n, void* stream) {
  if (!set) return fail(SOAX_E_ARG, "set is NULL");
  soax_status st;
  if ((st = check_n(set->L, n))) return st;
  const hipStream_t s = as_stream(stream);
  if ((st = ensure_capacity(set, n, s))) return st;
  if (n > set->n) {
    const int64_t add = n - set->n;
    ZeroArgs z{};
    auto part = [&](void* p, int64_t size) {
      z.base[z.parts] = static_cast<char*>(p) + set->n * size;
      z.bytes[z.parts++] = add * size;
    };
    if (has_soa(set))
      for (const Field& f : set->L.f)
        for (int c = 0; c < f.dim; ++c) part(set->soa[f.first_array + c], f.es);
    if (set->aos) part(set->aos, set->L.stride);
    HIP_TRY(launch_zero(z, s), "zero fill launch");
  }
  return set_size(set, n);
}

soax_status soax_push_back(soax_set* set, const void* host_records, int64_t count, void* stream) {
  if (!set) return fail(SOAX_E_ARG, "set is NULL");
  if (count < 0) return fail(SOAX_E_ARG, "count is negative");
  if (count > 0 && !host_records) return fail(SOAX_E_ARG, "host_records is NULL");
  soax_status st;
  if ((st = check_n(set->L, set->n + count))) return st;
  if (has_soa(set) && !set->owns && !set->soa_vec_ok)
    return fail(SOAX_E_LAYOUT, "push_back needs 16-byte aligned SoA arrays");
  const hipStream_t s = as_stream(stream);
  if ((st = ensure_capacity(set, set->n + count, s))) return st;
  if (count == 0) return SOAX_OK;
  const Layout& L = set->L;
  const int64_t n0 = set->n;
  const int64_t bytes = count * L.stride;
  {
    DevBuf stage, table;
    HIP_TRY(stage.alloc(bytes, s), "hipMallocAsync(staging)");
    HIP_TRY(hipMemcpyAsync(stage.p, host_records, bytes, hipMemcpyHostToDevice, s),
            "hipMemcpyAsync(records)");
    XposeArgs t = set->xpose_host;  // same fields; the appended range only
    if (has_soa(set)) {
      t.aos = static_cast<char*>(stage.p);
      t.n = count;
      t.stride = static_cast<int32_t>(L.stride);
      t.narrays = L.narrays;
      t.aligned = 1;
      for (const Field& f : L.f) {
        if (f.off % f.es || L.stride % f.es) t.aligned = 0;
        for (int c = 0; c < f.dim; ++c) {
          const int a = f.first_array + c;
          t.soa[a] = static_cast<char*>(set->soa[a]) + n0 * f.es;
          t.off[a] = static_cast<int32_t>(f.off + c * f.es);
          t.es[a] = f.es;
        }
      }
      group_by_size(t);
      HIP_TRY(table.alloc(sizeof(XposeArgs), s), "hipMallocAsync(table)");
      HIP_TRY(hipMemcpyAsync(table.p, &t, sizeof(XposeArgs), hipMemcpyHostToDevice, s),
              "hipMemcpyAsync(table)");
      HIP_TRY(launch_xpose(true, t, static_cast<const XposeArgs*>(table.p), s), "transpose launch");
    }
    if (set->aos)
      HIP_TRY(hipMemcpyAsync(set->aos + n0 * L.stride, stage.p, bytes, hipMemcpyDeviceToDevice, s),
              "hipMemcpyAsync(records)");
    // the host records and the host table must outlive the copies
    HIP_TRY(hipStreamSynchronize(s), "hipStreamSynchronize");
  }
  return set_size(set, n0 + count);
}

soax_status soax_rebind(soax_set* set, int64_t capacity, void* const* soa_ptrs, void* aos_ptr,
                        void* stream) {
  if (!set) return fail(SOAX_E_ARG, "set is NULL");
  if (set->owns) return fail(SOAX_E_STATE, "the set owns its buffers (use soax_reserve)");
  soax_status st;
  if ((st = check_n(set->L, capacity))) return st;
  if (capacity < set->n)
    return fail(SOAX_E_ARG, "capacity %lld is below n = %lld", static_cast<long long>(capacity),
                static_cast<long long>(set->n));
  if (has_soa(set) != (soa_ptrs != nullptr) || has_aos(set) != (aos_ptr != nullptr))
    return fail(SOAX_E_LAYOUT, "the new buffers must give the same copies as the old ones");
  if (capacity > 0 && soa_ptrs)
    for (int a = 0; a < set->L.narrays; ++a)
      if (!soa_ptrs[a]) return fail(SOAX_E_ARG, "soa_ptrs[%d] is NULL", a);
  const hipStream_t s = as_stream(stream);
  auto move = [&](void* dst, const void* src, int64_t bytes) {
    if (bytes == 0) return hipSuccess;
    if (aligned16(dst) && aligned16(src)) return launch_copy16(dst, src, bytes, s);
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, s);
  };
  if (set->n > 0) {
    if (soa_ptrs)
      for (const Field& f : set->L.f)
        for (int c = 0; c < f.dim; ++c) {
          const int a = f.first_array + c;
          HIP_TRY(move(soa_ptrs[a], set->soa[a], set->n * f.es), "copy into the new buffers");
        }
    if (aos_ptr)
      HIP_TRY(move(aos_ptr, set->aos, set->n * set->L.stride), "copy into the new buffers");
  }
  HIP_TRY(hipStreamSynchronize(s), "hipStreamSynchronize");  // copies done, old table unused
  if (soa_ptrs) set->soa.assign(soa_ptrs, soa_ptrs + set->L.narrays);
  set->aos = static_cast<char*>(aos_ptr);
  set->cap = capacity;
  set->aosoa = nullptr;  // the AoSoA table names the old SoA arrays
  ++set->generation;
  return finish_set(set);
}

soax_status soax_set_record(soax_set* set, int64_t i, const void* host_record) {
  if (!set || !host_record) return fail(SOAX_E_ARG, "set or host_record is NULL");
  if (i < 0 || i >= set->n) return fail(SOAX_E_ARG, "record %lld out of range", static_cast<long long>(i));
  const Layout& L = set->L;
  const char* in = static_cast<const char*>(host_record);
  if (set->aos)
    HIP_TRY(hipMemcpy(set->aos + i * L.stride, in, L.stride, hipMemcpyHostToDevice), "hipMemcpy");
  if (has_soa(set))
    for (const Field& f : L.f)
      for (int c = 0; c < f.dim; ++c)
        HIP_TRY(hipMemcpy(static_cast<char*>(set->soa[f.first_array + c]) + i * f.es,
                          in + f.off + c * f.es, f.es, hipMemcpyHostToDevice),
                "hipMemcpy");
  return SOAX_OK;
}

soax_status soax_remove_flagged(soax_set* set, const uint8_t* flags, int64_t* new_n, void* stream) {
  if (!set || !new_n) return fail(SOAX_E_ARG, "set or new_n is NULL");
  const int64_t n = set->n;
  if (n > 0 && !flags) return fail(SOAX_E_ARG, "flags is NULL");
  *new_n = n;
  if (n == 0) return SOAX_OK;
  const hipStream_t s = as_stream(stream);
  const int64_t tiles = container_tiles(n);
  if (!set->pinned_count)
    HIP_TRY(hipHostMalloc(reinterpret_cast<void**>(&set->pinned_count), sizeof(int32_t),
                          hipHostMallocDefault),
            "hipHostMalloc");
  // Tile counts and their exclusive sums, then the lists of moves: n / 2 moves
  // at most, or as many as a kept buffer has room for beside the counts.  More
  // than that take memory of their own once their number is known (4.1e6
  // moves and more; a second buffer on every call costs 4 to 8 us).
  DeviceScratch table, more;
  const size_t table_bytes = (2 * tiles * sizeof(int32_t) + 15) & ~size_t(15);
  const size_t list_bytes =
      std::min((2 * (n / 2) + 1) * sizeof(int32_t), DeviceScratch::kMaxBytes - table_bytes);
  HIP_TRY(table.take(table_bytes + list_bytes, s), "device memory for the counts and lists");
  int32_t* counts = static_cast<int32_t*>(table.get());
  int32_t* before = counts + tiles;
  HIP_TRY(launch_count_flags(flags, n, counts, before, set->pinned_count, s),
          "flag count launch");
  HIP_TRY(hipStreamSynchronize(s), "hipStreamSynchronize");  // the one wait: n' is returned
  const int64_t m = *set->pinned_count;
  const int64_t n_new = n - m;
  const int64_t moves_max = std::min(m, n_new);
  if (moves_max > 0) {
    MoveArgs mv{};
    int y = 0;
    const int sizes[3] = {8, 4, 1};
    for (int g = 0; g < 3; ++g) {
      if (has_soa(set))
        for (const Field& f : set->L.f)
          for (int c = 0; c < f.dim && f.es == sizes[g]; ++c)
            mv.base[y++] = static_cast<char*>(set->soa[f.first_array + c]);
      mv.group_end[g] = y;
    }
    if (set->aos) {
      mv.record = set->aos;
      mv.record_stride = static_cast<int32_t>(set->L.stride);
      mv.record_word = record_word(set);
    }
    const size_t need = (2 * moves_max + 1) * sizeof(int32_t);
    if (need > list_bytes) HIP_TRY(more.take(need, s), "device memory for the lists");
    int32_t* hole_at = need > list_bytes
                           ? static_cast<int32_t*>(more.get())
                           : reinterpret_cast<int32_t*>(static_cast<char*>(table.get()) + table_bytes);
    int32_t* mover_at = hole_at + moves_max;
    int32_t* nmoves = mover_at + moves_max;
    HIP_TRY(launch_rank_flags(flags, n, n_new, before, hole_at, mover_at, nmoves, s),
            "rank launch");
    HIP_TRY(launch_move_all(mv, hole_at, mover_at, nmoves, moves_max, s), "move launch");
  }
  *new_n = n_new;
  return set_size(set, n_new);
}

}  // extern "C"
