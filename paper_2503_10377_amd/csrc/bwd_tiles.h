// Tile and ring sizes of the wide bf16 backward kernels.
#pragma once

namespace sppo {

constexpr int kKvKeys = 128;  // keys per dK/dV workgroup (4 waves x 32)
constexpr int kDqRows = 128;  // query rows per dQ workgroup (4 waves x 32)
constexpr int kSB = 32;       // rows (dK/dV) or keys (dQ) per sub-block
constexpr int kRing = 6;      // LDS ring slots
constexpr int kAhead = 5;     // sub-blocks loaded ahead of the one in use
// Each step's barrier also waits for sub-block n+2, so the B phase of step n
// can read A(n+1)'s first natural operands in its last MFMA slots (which read
// nothing else), and A's last slots read B's first transposed operands.
static_assert(kAhead == kRing - 1, "a slot is refilled right after its last reader");

}  // namespace sppo
