// Single-launch small solves for wires of 20 segments (19 rooftop unknowns).
#define CHAFF_KNB 19
#define CHAFF_KNS kr19
#include "krylov_small.hpp"
