// Shares of the chip for launches whose workgroups wait for each other.
//
// Such a launch needs all its workgroups resident at once, so a small kernel before it claims room on the device and
// waits until there is some; the last kernel of the group (or the last workgroup out) gives the claim back.  The launches
// of a group are queued together, under resident_launches(): a kernel that waits for room never stands between another
// group's launches where streams share a hardware queue.
//
// What is counted: shares of 32 workgroups -- workgroups go to the 8 dies in turn and, on a die, to its 4 shader engines,
// so a share is at most one workgroup per engine (8 compute units) and the sums hold for every engine, not only for the
// chip.  A full claim counts on a compute unit of its own per workgroup; of a light one a unit holds three, as long as no full
// claim is about.  Any placement of the workgroups then leaves room for those still to come.
//
// The waves that wait for room must not sit where a grid that has its room still has to go: beside the waves that a claim may
// put on a SIMD there must be room, in its 512 registers, for four waiting ones of 8, as many as a process has hardware
// queues.  Full claims: amq_seqw.hip and amq_seqw_tiles.hip with two waves per SIMD of at most kResidentRegisters, and the forms
// of amq_seq1_body.h that are not light, with one of at most 256.  Light claims: amq_lstm_seqg.hip (up to 144 registers) and
// the forms of amq_seq1_body.h for 513 to 1024 units (up to 160), with one wave per SIMD and workgroup.
//
// The word on the device: full shares in bits 0..7, light ones in bits 8..15, and the door.  Whoever finds no room closes
// the door and is the next to get some; small claims do not keep a large one waiting for ever.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

namespace amq {

constexpr int kShareGrid = 32;
constexpr int kLightPerUnit = 3;
constexpr int kResidentRegisters = 240;  // (the attribute that limits them counts half: one of the two kinds)
constexpr unsigned kDoor = 1u << 31;

struct ResidentClaim {
  unsigned* word;            // null: no room is counted on this device
  unsigned mine;             // full shares, or light shares << 8
  unsigned shares;           // shares of the device
  unsigned long long ticks;  // of the 100 MHz clock: how long to wait for room
};
ResidentClaim resident_claim(long long grid, bool light);
std::mutex& resident_launches();

__device__ __forceinline__ bool resident_room(unsigned used, const ResidentClaim& c) {
  const unsigned sum = (used & ~kDoor) + c.mine, full = sum & 255u, light = sum >> 8;
  return full ? full + light <= c.shares : light <= kLightPerUnit * c.shares;
}
// To be called by one lane.  (What it reads goes to the scalar unit: a wave that waits here should hold few registers.)
__device__ __forceinline__ bool take_resident_share(const ResidentClaim& c) {
  if (!c.word) return true;
  const unsigned long long start = wall_clock64();
  unsigned used = 0u, door = 0u;  // door: set once it is this claim that holds it
  for (;;) {
    // (the common case is an idle chip: one exchange)
    unsigned next = used;
    if ((used & kDoor) == door) next = resident_room(used, c) ? (used & ~kDoor) + c.mine : used | kDoor;
    if (next != used) {
      unsigned seen = used;
      __hip_atomic_compare_exchange_strong(c.word, &seen, next, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((unsigned)__builtin_amdgcn_readfirstlane((int)seen) == used) {
        if (!(next & kDoor)) return true;
        door = kDoor;
      }
    }
    if (wall_clock64() - start > c.ticks) {
      if (door) __hip_atomic_fetch_and(c.word, ~kDoor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
    if (next == used || (next & kDoor)) __builtin_amdgcn_s_sleep(32);
    used = (unsigned)__builtin_amdgcn_readfirstlane(
        (int)__hip_atomic_load(c.word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  }
}
__device__ __forceinline__ void give_resident_share(const ResidentClaim& c) {
  if (c.word) __hip_atomic_fetch_sub(c.word, c.mine, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}
// Test hook: takes (or with a negative number gives back) full shares without waiting.
hipError_t launch_hold_shares(int shares, hipStream_t s);
// Test hook: writes the word to `room`.
hipError_t launch_read_shares(unsigned* room, hipStream_t s);

}  // namespace amq
