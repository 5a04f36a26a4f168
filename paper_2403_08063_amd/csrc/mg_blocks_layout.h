// Constants of the 2:1 refined layout's face table and ghost-plane array.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

constexpr int kBlocks = 120;
// per block and face: kind, neighbour blocks[4], quadrant s1, s2, slot (see build_faces)
constexpr int kFaceInts = 8;
enum { kFaceBoundary = 0, kFaceSame = 1, kFaceF2C = 2, kFaceC2F = 3 };

// Place of ghost (t1, t2) (1 .. B, first tangential axis fastest) of a block's face in an array
// that holds the layout's ghost planes alone.
__device__ __forceinline__ size_t ghost_index(int B, int b, int face, int t1, int t2)
{
  return (((size_t)b * 6 + face) * B + (t2 - 1)) * (size_t)B + (t1 - 1);
}
