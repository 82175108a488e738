// How a small grid's update set is split over the chip for a whole time loop in
// one launch.  Plain C++: the host and its tests use it without HIP.
#pragma once

namespace emm {

constexpr int kResPlanes = 5;         // planes per thread at most
// threads per tile at most: 128 registers each hold one plane, more take 256
constexpr int resident_threads(int planes) { return planes == 1 ? 1024 : 512; }
// words a thread receives per half step at most
constexpr int resident_words(int planes) { return planes == 1 ? 8 : 12; }
constexpr int kResTall = 32;          // planes per tile at most
constexpr int kResSlot = 6200;        // floats of one field component's tile in LDS
constexpr int kResRows = 192;         // sampled rows per tile and half step at most

// The split of a grid's update set into gy x gz tiles of whole x rows, one
// per compute unit; a tile's planes go to groups of `planes` planes.
struct ResidentPlan {
    int gy = 0, gz = 0;               // 0: the grid does not qualify
    int ty = 0, tz = 0;               // largest tile: rows, planes
    int planes = 0, groups = 0;       // planes per thread, thread groups
    int threads = 0;
};

// Plan for a padded grid, or gy = 0.  cus: compute units of the device.
ResidentPlan resident_plan(int r, int n1, int n2, int n3, int cus);

// The highest element of the block's six component tiles (E then H, kResSlot
// floats each, one after another) that a thread reads: taps of H, whose tiles
// come last.  The last thread group may reach past the tile's last plane; what
// it computes there is not stored, but its taps still read, across the tiles
// that follow.  Plans keep this below 6 kResSlot.
inline long resident_reach(int r, int n1, const ResidentPlan &p) {
    const int L = 2 * r, end = p.groups * p.planes;                // planes of all groups
    const long zs = (long)(p.ty + L - 1) * n1;
    const long cell = (long)(p.ty - 1 + r) * n1 + n1 - 1 - r;       // last column, in its LDS plane
    const long y = cell + (long)(r - 1) * n1, x = cell + r - 1;     // last taps of component 3
    const long xy = 5l * kResSlot + (end - 1 + r) * zs + (y > x ? y : x);
    const long z = 4l * kResSlot + (end - 1 + L - 1) * zs + cell;   // the z column of component 2
    return xy > z ? xy : z;
}

}  // namespace emm
