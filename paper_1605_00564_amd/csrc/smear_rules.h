// How Gaussian smearing splits its vectors over two kernels.  Plain C++, shared by
// the smearing and a CPU test.
#pragma once

namespace dfl {

// Groups of four among n vectors of V sites; the others take the kernel of one vector
// at a time.  With vectors left over, a step is two launches, which small lattices
// feel (ten steps, FP64, us, split / all by one: V = 4096: n = 5 138 / 76, n = 13
// 159 / 93; 16384: 175 / 146, 330 / 319; 32768: 257 / 253, 596 / 593; 65536:
// n = 5 492 / 500, n = 13 1213 / 1420).  Without any the groups are as fast or faster
// from 4 vectors of 256 sites on.
inline int gauss_groups(long V, int n) { return n % 4 && V <= 32768 ? 0 : n / 4; }

}  // namespace dfl
