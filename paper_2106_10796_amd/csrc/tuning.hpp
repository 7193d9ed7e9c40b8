// Build-time knobs of the kernels (launch shapes, cache policy); the defaults are the measured best.
#pragma once

// Cache policy is chosen by measurement on MI355X; each kernel states its own launch shape.
// Non-temporal loads and stores are worth about 15 % (every byte is touched once
// per step, so nothing should stay in L2 or the memory-side cache).
#ifndef CDSGD_NT
#define CDSGD_NT 1
#endif
#ifndef CDSGD_NT_LOAD
#define CDSGD_NT_LOAD CDSGD_NT
#endif
#ifndef CDSGD_NT_STORE
#define CDSGD_NT_STORE CDSGD_NT
#endif
#ifndef CDSGD_XCD_FULL
#define CDSGD_XCD_FULL 0
#endif
#ifndef CDSGD_XCD_PIECES
#define CDSGD_XCD_PIECES 1
#endif
#ifndef CDSGD_FULL_BLOCK
#define CDSGD_FULL_BLOCK 64
#endif
