// trace_lds.h -- what a workgroup of the traversal kernels keeps in LDS, and
// where.  Plain C++: the kernels take their pointers from here, the launch
// its bytes, and the layout can be checked on the host.
//
// A workgroup runs one of two paths, the same for all its waves:
//  - a ray per lane: lds_depth stack entries per thread (entry e of thread t
//    at word e * kThreads + t), then a staging ring per wave;
//  - a group of W lanes per ray: kStackCap stack entries per group, from the
//    first word on, and no ring.
// The two overlay each other, so a wave touches nothing of the one path
// before it knows that its workgroup does not run the other: no barrier
// stands between the waves of a workgroup.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace rgt {

constexpr int kThreads = 256;     // threads per workgroup of the trace kernels
constexpr int kMaxLdsStack = 32;  // most stack entries per lane kept in LDS (chosen per launch)
constexpr int kPrivStack = 96;    // further entries per lane in private memory
constexpr int kStackCap = 8 + kPrivStack;  // guaranteed capacity (at the smallest LDS depth, 8)

// Packets in a wave's staging ring; a ring holds K result words per ray and
// packet, then per packet a mask (8 bytes), an owner and a packet number.
constexpr int kStageSlots = 4;

// Bytes of one wave's staging ring.
constexpr size_t ring_bytes(int K) { return (size_t)kStageSlots * (K * 64 * 4 + 16); }
// Where the ring of wave `wave` of the workgroup starts.
constexpr size_t ring_at(int K, int lds_depth, int wave) {
    return (size_t)lds_depth * kThreads * 4 + (size_t)wave * ring_bytes(K);
}
// Bytes of a workgroup that runs a ray per lane.
constexpr size_t lanes_bytes(int K, int lds_depth) { return ring_at(K, lds_depth, kThreads / 64); }

// Where the stacks of the groups of wave `wave` start (groups of W lanes).
constexpr size_t group_stacks_at(int W, int wave) { return (size_t)wave * (64 / W) * kStackCap * 4; }
// Bytes of a workgroup that runs a group of lanes per ray.
constexpr size_t groups_bytes(int W) { return group_stacks_at(W, kThreads / 64); }

}  // namespace rgt
