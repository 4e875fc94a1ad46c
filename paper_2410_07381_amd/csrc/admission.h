// Which of the best-effort clients that wait is put on the GPU next.  Plain C++: nothing here knows a GPU.
#pragma once
#include <stdint.h>

namespace tally {

// What workgroups occupy of a compute unit: LDS bytes, waves, registers per lane of a SIMD.
struct Demand {
  uint32_t lds, waves, regs;
};

// A kernel is put on the GPU only if all the workgroups it brings fit beside the
// best-effort workgroups already resident: a dispatch that waits for resources blocks
// its hardware pipe for every queue mapped to that pipe, the high-priority queue
// possibly among them (two 128 KB-LDS GEMMs launched together held high-priority
// kernels back for milliseconds).  Clients that have to wait are served first come,
// first served.  A client with the GPU to itself is always admitted.
//
// Client has `ticket` (its place in the queue, 0 while it is not waiting) and `resident` (a Demand).  enter() is
// asked last, once client c may go: true, and it is in; false, something else came between, and it waits on in its
// place.
template <class Client, class Enter>
bool admit(Client *clients, uint32_t n, uint32_t c, const Demand &d, uint32_t lds_per_cu, uint64_t *last_ticket, Enter enter) {
  Client &cl = clients[c];
  if (cl.ticket == 0) cl.ticket = ++*last_ticket;
  uint32_t lds = 0, waves = 0, regs = 0, others = 0;
  for (uint32_t o = 0; o < n; ++o) {
    if (o == c) continue;
    const Client &oc = clients[o];
    if (oc.ticket != 0 && oc.ticket < cl.ticket) return false;
    if (oc.resident.waves) others++;
    lds += oc.resident.lds;
    waves += oc.resident.waves;
    regs += oc.resident.regs;
  }
  // (one wave slot and 32 registers are kept back for the newcomer's relay)
  if (others && (lds + d.lds > lds_per_cu || waves + d.waves > 31u || regs + d.regs > 480u)) return false;
  if (!enter()) return false;
  cl.ticket = 0;
  return true;
}

}  // namespace tally
