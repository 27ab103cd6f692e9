// hb_internal.hpp -- host-side declarations shared by the libhb translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

namespace hb {

// Thread-local last-error text (exposed by hb_last_error) and the status it goes with.
int set_error(int status, const std::string &msg);
int hip_error(hipError_t e, const char *what);

// Fixed-length batch (hb_kernels.hip): message i at i * fixed_len, one lane per message in
// index order, digest i at out + i * stride.  Returns the hipError_t of the launch.
hipError_t launch_fixed(int algo, const uint8_t *msgs, uint64_t n, uint64_t fixed_len, uint8_t *out, uint32_t stride,
                        hipStream_t stream);

// As launch_fixed for packed digests, by chain pairs (hb_ragged.hip), for the batches that
// fixed_chain_applies to: few messages.  staged: the other way would stage them through LDS.
bool fixed_chain_applies(int algo, uint64_t n, uint64_t len, bool staged);
hipError_t launch_fixed_chain(int algo, const uint8_t *msgs, uint64_t n, uint64_t len, uint8_t *out, hipStream_t stream);

int digest_size(int algo);

// SIMDs of the current device (four per CU).
uint32_t device_simds();

// Packed batch of any lengths in one launch, without workspace (hb_ragged.hip): message i's
// digest at out + i * stride.  algos non-null: per-message ids (unknown ones give an all-zero
// slot), else every message uses algo.
hipError_t launch_ragged(const uint8_t *algos, int algo, const uint8_t *msgs, const uint64_t *offs, const uint64_t *lens,
                         uint64_t n, uint8_t *out, uint32_t stride, hipStream_t stream);

// One lane per message for n messages makes at most one wave per SIMD of the current
// device: every wave runs alone, so the compression with the fewest instructions is the
// faster one; from two waves on a SIMD the one ordered for sharing is (hb_issue.hpp).
bool few_waves(uint64_t n);

// Hash messages [i0, i1) on host threads (the CPU share of a CPU + GPU split); message i's
// digest goes to out + (i - i0) * stride.  threads <= 0: all hardware threads.
void cpu_hash_range(const uint8_t *algos, int algo, const uint8_t *msgs, const uint64_t *offs, const uint64_t *lens,
                    uint64_t i0, uint64_t i1, uint8_t *out, uint32_t stride, int threads);

// Copy `bytes` between device-accessible buffers with a kernel on `stream` (no copy
// engine): device memory, or pinned host memory through its device mapping.
hipError_t launch_copy(void *dst, const void *src, uint64_t bytes, hipStream_t stream);

struct ServeRings;

// The resident serving kernel (hb_serve.hip): `workgroups` workgroups of 256 lanes, the
// first wave dispatching, the rest hashing published items until told to stop or idle.
hipError_t launch_serve(const ServeRings &rings, uint32_t gen, int workgroups, hipStream_t stream);

// The paper's 9-digit decimal workload, generated on the device (see hash_digits9).
hipError_t launch_digits9(int algo, uint64_t start, uint64_t n, uint8_t *out, hipStream_t stream);

}  // namespace hb
