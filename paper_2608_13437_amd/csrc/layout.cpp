// What fixes the update's memory traffic besides its kernels: the population
// layout (region stride) and the default launch shape of each storage type.
#include <hip/hip_runtime.h>

#include "../../include/cnsf.h"
#include "api_common.h"
#include "cnsf_impl.h"
#include "launch.h"

namespace cnsf {

Launch default_launch(int storage) {
  // Measured on the 512^3 update with the grouped slot layout: one block per
  // tile throughout; 256-cell tiles dealt to the XCDs in contiguous spans for
  // FP32 and BF16, 512-cell tiles in hardware order for FP16.
  Launch lc;
  lc.block = 256;
  lc.tile = 256;
  lc.grid = 0;
  lc.remap = 1;
  if (storage == CNSF_STORAGE_FP16) {
    lc.tile = 512;
    lc.remap = 0;
  }
  return lc;
}

// Up to 96 x 1024 cells 64-cell blocks: what such an update costs is latency, and 256-cell blocks leave CUs
// without work (us per update, 256 -> 64 cells: FP32 16^3 5.3 -> 4.2, 24^3 5.8 -> 4.7, 32^3 6.9 -> 6.3, 40^3
// equal, 46^3 12.5 -> 12.4, but 48^3 13.7 -> 14.1; BF16 24^3 5.4 -> 4.9, 32^3 5.8 -> 5.5).  FP16 lattices
// that the 256 MB last-level cache holds do not want the order of the large ones: 256-cell tiles in spans
// (512-cell tiles in hardware order / in spans / 256-cell tiles: 48^3 10.8 / 10.2 / 8.6, 56^3 15.6 / 14.4 / 13.2,
// 80^3 37.0 / 35.3 / 34.3, 100^3 71.2 / 68.6 / 63.0, but 128^3 163 against 179), except where 256-cell tiles
// would be three to four blocks per CU: the fullest CU has the same cells then, and half the blocks to start
// (58^3, 2.98 blocks per CU, 17.1 / 15.4 / 15.0; 59^3 17.7 / 16.5 / 16.6; 60^3 17.9 / 17.2 / 17.2; 61^3 18.4 / 17.2 /
// 17.1; 62^3 19.0 / 18.1 / 18.5; 63^3 19.6 / 19.0 / 19.2; 64^3, 4.0, 18.6 / 18.5 / 19.1; 65^3, 4.2, 24.3 / 23.7 / 21.7;
// 66^3 24.6 / 24.0 / 22.0; 68^3 25.3 / 24.7 / 23.1).
Launch lattice_launch(int storage, uint64_t ncells, int cus) {
  Launch lc = default_launch(storage);
  if (ncells <= 96 * 1024) {
    lc.block = 64;
    lc.tile = 64;
    lc.remap = 1;
  } else if (storage == CNSF_STORAGE_FP16 && (uint64_t)NP * 2 * ncells <= 256000000ull) {
    const uint64_t blocks = (ncells + 255) / 256;
    if (blocks <= 3ull * cus || blocks > 4ull * cus) lc.tile = 256;
    lc.remap = 1;
  }
  return lc;
}

// Elements between consecutive component regions: 7 slots of the cell count
// rounded up to whole slot groups.
uint64_t component_stride(uint64_t ncells, int storage) {
  (void)storage;
  return (uint64_t)NV * ((ncells + SLOT_GROUP - 1) / SLOT_GROUP * SLOT_GROUP);
}

}  // namespace cnsf
