// Where the single-launch Cholesky factorisation (chol_chain_kernel) puts its near-diagonal tasks: pure integer arithmetic, which the
// model of its schedule in the tests is compared with.
#pragma once

namespace dion {

struct NearOrder {
  bool far;
  int shift;   // helper workgroup g of pr * pc has place (g + shift) mod (pr * pc), counted from the other end if far
};
// Workgroup that the near-diagonal tasks of row 0 start at, those of the next rows following from there, three to a row: at the
// front, at the far end in falling order, or (shift) in between.  The other tiles fill the workgroups from the front, row by
// row, once per whole round of 2 pr rows; `beyond` workgroups hold the rows after the last whole round as well.
//   less than a round: where all near-diagonal tasks and all other tiles have room side by side the former go to the far end, else
//     to the front, whose rows are through first: 8 panels on 7 x 9 70 / 83 us, 16 on 15 x 17 138 / 150, 24 on 15 x 17 289 /
//     240, 32 403 / 357 (far end / front).
//   a round and more, a workgroup for every task: behind the `beyond` ones, where these would get two fifths of the tasks and more:
//     36 panels on 15 x 17 468 / 437, 40 601 / 556, 44 750 / 676, 48 840 / 768, 52 947 / 925, 20 on 7 x 9 279 / 273;
//     below that the front: 16 on 7 x 9 190 / 201 (front / behind).
//   more tasks than workgroups: far end, where the last rows' second tasks then lie beside no row beyond the round: 23 panels on
//     7 x 9 382 / 368, 25 444 / 408, 31 698 / 665, 33 822 / 746, without such room 26 459 / 484, 28 541 / 567 (front / far end).
//     On 3 x 5 the front: 7 panels 81 / 86, 13 246 / 251.
constexpr NearOrder near_order(int nb, int pr, int pc) {
  const int groups = pr * pc, round = 2 * pr, tasks = 3 * nb, beyond = ((nb % round) * pc + 1) / 2;
  const bool far = beyond > 0 && (nb < round ? tasks + beyond <= groups
                                             : groups >= 63 && tasks > groups && tasks < 2 * groups && tasks - groups + beyond <= groups);
  const bool behind = nb > round && tasks <= groups && 5 * beyond >= 2 * tasks;
  return NearOrder{far, behind ? groups - beyond : 0};
}

}  // namespace dion
