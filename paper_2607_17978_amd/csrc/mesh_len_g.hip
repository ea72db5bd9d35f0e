// Mesh passes of the axis lengths of group g (mesh_len.h).
#include "mesh_len_launch.h"

#define LENGTHS(X) X(24) X(48) X(128) X(300) X(360)
QEQ_LEN_GROUP(mesh_len_g, LENGTHS)
